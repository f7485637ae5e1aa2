// Kurganov-Tadmor central scheme (Sec. 3.2, eqs. (5)-(8)) on gfx950.
//
// One step = two stages of the Runge-Kutta midpoint rule,
//   U* = U^n + dt/2 L(U^n),   U^{n+1} = U^n + dt L(U*)   (+ the external kick),
// L = -(dH_x/dx + dH_y/dy) with the local-speed flux of eq. (6) at faces
// reconstructed by component-wise MC-limited linear primitive profiles.  On a
// 2-D grid both stages run in one launch with the work decomposition of the
// characteristic sweep (a wavefront per column strip marching up rows, x
// neighbours by DPP lane shifts, y neighbours from row register sets), U* living
// in registers (large grids) or in LDS; a 1-D grid takes one launch per stage.
// The kernels carry half slopes (face states w -+ h) and twice the flux (the
// update coefficients take the 1/2).
#include <algorithm>
#include <cstdlib>

#include "csh_device.h"
#include "csh_internal.h"
#include "csh_xcd.h"

namespace csh {

template <typename T>
__device__ __forceinline__ double kt_dt(const StepArgs<T>& p, double* t_now)
{
    const Slot& sl = p.slots[p.s_in];
    *t_now = sl.t;
    if (p.dt_in) return *p.dt_in;
    if (!p.dev_dt) return p.dt;
    double dt = p.cfl / slot_rate(sl);
    if (p.t_end > 0.0) {
        if (sl.t >= p.t_end) dt = 0.0;
        else if (sl.t + dt > p.t_end) dt = p.t_end - sl.t;
    }
    return dt;
}

// 1-D grids: one launch per stage, a wavefront per 60 cells (2 halo lanes per
// side); the first stage records the step's timestep in its input slot for
// the second
template <typename T, bool FINAL>
__global__ __launch_bounds__(64 * kWaves) void kt_kernel(StepArgs<T> p)
{
    double t_now;
    const double dt = kt_dt(p, &t_now);
    if (FINAL && blockIdx.x == 0) slot_clear(p.slots[p.s_reset], threadIdx.x);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (!FINAL) {
            p.slots[p.s_in].dt = dt;
        } else {
            p.slots[p.s_out].t = t_now + dt;
            if (p.dt_log) *p.dt_log = dt;
        }
    }
    const int lane = threadIdx.x & 63;
    const int wid = blockIdx.x * kWaves + wave_in_block();
    if (wid >= p.nstrips) return;  // uniform per wavefront
    const int c = wid * kStrip - 2 + lane;
    const int gc = map_index(c, p.nx, p.bcx);
    const bool own = lane >= 2 && lane < 2 + kStrip && c < p.nx;
    const double h = FINAL ? dt : 0.5 * dt;  // stage length
    const T cx = T(0.5 * h / p.dx);  // the flux below is 2H
    const Planes<T> in(p.U, (size_t)p.nx);
    const OutPlanes<T> out(p.Unew, (size_t)p.nx);
    const Cons<T> C0 = in.load((unsigned)gc);
    const Prim<T> W0 = to_prim(C0);
    const Prim<T> s = mc_half_slope(lane_shift<-1>(W0), W0, lane_shift<+1>(W0));
    const Cons<T> F = kt_flux2_x(plus(W0, s), lane_shift<+1>(sub(W0, s)));
    const Cons<T> Fm = lane_shift<-1>(F);
    Cons<T> Un = update(FINAL ? Planes<T>(p.Ubase, (size_t)p.nx).load((unsigned)gc) : C0, cx, F, Fm);
    double smax = 0.0;
    bool bad = false;
    if (FINAL) kick(Un, p, dt, c, 0, false);
    if (own) {
        out.store((unsigned)c, Un);
        if (FINAL) {
            smax = fmax(smax, checked_rate<T, false>(Un, 1.0 / p.dx, 0.0, bad));
        }
    }
    if (FINAL) {
        smax = wave_max(smax);
        if (lane == 0) slot_add(p.slots[p.s_out], blockIdx.x, smax);
        if (__any(bad) && lane == 0) raise_flag(p.flag);
    }
}

// ---- both stages in one launch (2-D) ---------------------------------------------------------
//
// The first stage's result U* is never stored: each wavefront forms the U*
// rows its second stage needs and keeps them, in primitive form, in a ring of
// three row register sets.  Stage 1 marches rows y0-3 .. y1+2 (U* rows y0-2 ..
// y1+1, the second stage's stencil) and stage 2 follows two rows behind it, so
// a step reads U^n once (a wavefront keeps its last four input rows in LDS for
// the base of stage 2) and writes U^{n+1} once: 96 B per cell-update instead of
// the 240 B of two launches.  A wavefront owns 56 columns: stage 1 is valid on
// lanes 2..61, stage 2 on lanes 4..59.
//
// Boundaries.  The boundary conditions apply to U* as to any state: at a
// ghost position stage 2 sees U* of the mapped cell.  With periodic
// boundaries the lanes and rows of a wavefront hold a contiguous window of
// the torus, so its own U* at a ghost position is already that value; with
// outflow boundaries the ghost columns take U* of the edge column by a lane
// read, and the ghost rows a copy of the edge row.

constexpr int kFusedStrip = 56;  // owned columns per wavefront of the fused step

template <typename T>
__global__ __launch_bounds__(64 * kWaves) void kt_fused_kernel(StepArgs<T> p)
{
    double t_now;
    const double dt = kt_dt(p, &t_now);
    if (blockIdx.x == 0) {
        slot_clear(p.slots[p.s_reset], threadIdx.x);
        if (threadIdx.x == 0) {
            p.slots[p.s_out].t = t_now + dt;
            if (p.dt_log) *p.dt_log = dt;
        }
    }
    const int lane = threadIdx.x & 63;
    const int wid = blockIdx.x * kWaves + wave_in_block();
    if (wid >= p.nstrips * p.nsegs) return;  // uniform per wavefront
    const int sx = wid % p.nstrips, sy = wid / p.nstrips;
    const int c0 = sx * kFusedStrip - 4;  // column of lane 0
    const int c = c0 + lane;
    const int gc = map_index(c, p.nx, p.bcx);
    const bool own = lane >= 4 && lane < 4 + kFusedStrip && c < p.nx;
    // outflow in x: ghost lanes read U* from the lane of the edge column
    const bool xfix = p.bcx != 0 && (c0 < 0 || c0 + 63 >= p.nx);
    const int src = c < 0 ? -c0 : (c >= p.nx ? p.nx - 1 - c0 : lane);
    const size_t plane = (size_t)p.nx * p.ny;
    const double h1 = 0.5 * dt;  // stage lengths; the fluxes below are 2H
    const T cx1 = T(0.5 * h1 / p.dx), cy1 = T(0.5 * h1 / p.dy);
    const T cx2 = T(0.5 * dt / p.dx), cy2 = T(0.5 * dt / p.dy);
    const double idx = 1.0 / p.dx, idy = 1.0 / p.dy;
    const Planes<T> in(p.U, plane);
    const OutPlanes<T> out(p.Unew, plane);
    double smax = 0.0;
    bool bad = false;
    const int y0 = sy * p.ty, y1 = min(y0 + p.ty, p.ny);
    const int a1 = y0 - 2, b1 = y1 + 2;  // U* rows formed here: [a1, b1)
    auto load_row = [&](int r) -> Cons<T> { return in.load((unsigned)(map_index(r, p.ny, p.bcy) * p.nx + gc)); };
    auto fix_x = [&](const Prim<T>& w) -> Prim<T> {
        if (!xfix) return w;
        return {__shfl(w.r, src, 64), __shfl(w.u, src, 64), __shfl(w.v, src, 64), __shfl(w.pxx, src, 64),
                __shfl(w.pxy, src, 64), __shfl(w.pyy, src, 64)};
    };

    // the U^n rows of the last four iterations in LDS, for the base of stage 2
    // (each lane reads and writes only its own column: no barrier)
    __shared__ T ring_lds[kWaves][4][6][64];
    T(*const ring)[6][64] = ring_lds[wave_in_block()];
    auto ring_put = [&](int r, const Cons<T>& U) {
        T(*const q)[64] = ring[(r - y0) & 3];
        q[0][lane] = U.r;
        q[1][lane] = U.mx;
        q[2][lane] = U.my;
        q[3][lane] = U.exx;
        q[4][lane] = U.exy;
        q[5][lane] = U.eyy;
    };
    auto ring_get = [&](int r) -> Cons<T> {
        const T(*const q)[64] = ring[(r - y0) & 3];
        return {q[0][lane], q[1][lane], q[2][lane], q[3][lane], q[4][lane], q[5][lane]};
    };

    Cons<T> Ca = load_row(y0 - 4), Cb = load_row(y0 - 3), Cc = load_row(y0 - 2);
    Prim<T> Wa = to_prim(Ca), Wb = to_prim(Cb), Wc = to_prim(Cc);
    ring_put(y0 - 4, Ca);
    ring_put(y0 - 3, Cb);
    ring_put(y0 - 2, Cc);
    Prim<T> Sa{}, Sb{}, Sc{};  // U* rows (primitive)
    Prim<T> yhi1{}, yhi2{};
    Cons<T> acc1{}, acc2{};

    // stage 1 at row r: Wm, W0, Wp rows r-1, r, r+1 of U^n (Wm refilled with
    // row r+2), C0 row r conserved (Cm refilled); finishes U* row r-1 into Sn
    // (Sm3, Sm2: the ring's rows r-3, r-2)
    auto stage1 = [&](int r, Prim<T>& Wm, const Prim<T>& W0, const Prim<T>& Wp, Cons<T>& Cm, const Cons<T>& C0,
                      Prim<T>& Sn, Prim<T>& Sm3, Prim<T>& Sm2) {
        const Cons<T> Unext = load_row(r + 2);
        const Prim<T> sxv = mc_half_slope(lane_shift<-1>(W0), W0, lane_shift<+1>(W0));
        const Prim<T> syv = mc_half_slope(Wm, W0, Wp);
        if (r >= a1) {
            const Cons<T> G = swap(kt_flux2_x(swap(yhi1), swap(sub(W0, syv))));  // face r - 1/2
            if (r > a1) {
                if (p.bcy != 0 && r - 1 >= p.ny) {
                    Sn = Sm2;  // outflow: the ghost rows above copy row ny - 1
                } else {
                    Sn = fix_x(to_prim(Cons<T>{acc1.r - cy1 * G.r, acc1.mx - cy1 * G.mx, acc1.my - cy1 * G.my,
                                               acc1.exx - cy1 * G.exx, acc1.exy - cy1 * G.exy,
                                               acc1.eyy - cy1 * G.eyy}));
                    if (p.bcy != 0 && r - 1 == 0) Sm2 = Sm3 = Sn;  // outflow: the ghost rows below copy row 0
                }
            }
            if (r < b1) {
                const Cons<T> F = kt_flux2_x(plus(W0, sxv), lane_shift<+1>(sub(W0, sxv)));
                const Cons<T> Fm = lane_shift<-1>(F);
                acc1 = {C0.r - cx1 * (F.r - Fm.r) + cy1 * G.r,         C0.mx - cx1 * (F.mx - Fm.mx) + cy1 * G.mx,
                        C0.my - cx1 * (F.my - Fm.my) + cy1 * G.my,     C0.exx - cx1 * (F.exx - Fm.exx) + cy1 * G.exx,
                        C0.exy - cx1 * (F.exy - Fm.exy) + cy1 * G.exy, C0.eyy - cx1 * (F.eyy - Fm.eyy) + cy1 * G.eyy};
            }
        }
        yhi1 = plus(W0, syv);
        Wm = to_prim(Unext);
        Cm = Unext;
        ring_put(r + 2, Unext);  // into the slot of row r - 2, read before this
    };

    // stage 2 at row q on U* rows q-1, q, q+1; B = row q of U^n
    auto stage2 = [&](int q, const Prim<T>& Wm, const Prim<T>& W0, const Prim<T>& Wp, const Cons<T>& B) {
        const Prim<T> sxv = mc_half_slope(lane_shift<-1>(W0), W0, lane_shift<+1>(W0));
        const Prim<T> syv = mc_half_slope(Wm, W0, Wp);
        if (q >= y0) {
            const Cons<T> G = swap(kt_flux2_x(swap(yhi2), swap(sub(W0, syv))));  // face q - 1/2
            if (q > y0) {
                Cons<T> Un = {acc2.r - cy2 * G.r,     acc2.mx - cy2 * G.mx,   acc2.my - cy2 * G.my,
                              acc2.exx - cy2 * G.exx, acc2.exy - cy2 * G.exy, acc2.eyy - cy2 * G.eyy};
                kick(Un, p, dt, c, q - 1, true);
                if (own) {
                    out.store((unsigned)((q - 1) * p.nx + c), Un);
                    smax = fmax(smax, checked_rate(Un, idx, idy, bad));
                }
            }
            if (q < y1) {
                const Cons<T> F = kt_flux2_x(plus(W0, sxv), lane_shift<+1>(sub(W0, sxv)));
                const Cons<T> Fm = lane_shift<-1>(F);
                acc2 = {B.r - cx2 * (F.r - Fm.r) + cy2 * G.r,         B.mx - cx2 * (F.mx - Fm.mx) + cy2 * G.mx,
                        B.my - cx2 * (F.my - Fm.my) + cy2 * G.my,     B.exx - cx2 * (F.exx - Fm.exx) + cy2 * G.exx,
                        B.exy - cx2 * (F.exy - Fm.exy) + cy2 * G.exy, B.eyy - cx2 * (F.eyy - Fm.eyy) + cy2 * G.eyy};
            }
        }
        yhi2 = plus(W0, syv);
    };

    // one row of the march: stage 1 at r, then stage 2 at q = r - 2 (from the
    // first row whose stencil stage 1 has finished); S0, Sr3, Sr2: the ring
    // slots of U* rows r-1, r-3, r-2
    auto iter = [&](int r, Prim<T>& Wm, const Prim<T>& W0, const Prim<T>& Wp, Cons<T>& Cm, const Cons<T>& C0,
                    Prim<T>& S0, Prim<T>& Sr3, Prim<T>& Sr2) {
        const int q = r - 2;
        const Cons<T> B = ring_get(q);  // row q's U^n (used for q in [y0, y1) only)
        stage1(r, Wm, W0, Wp, Cm, C0, S0, Sr3, Sr2);
        if (q >= y0 - 1) stage2(q, Sr3, Sr2, S0, B);
    };

    for (int r = a1 - 1; r <= b1; r += 3) {
        iter(r, Wa, Wb, Wc, Ca, Cb, Sa, Sb, Sc);
        if (r + 1 > b1) break;
        iter(r + 1, Wb, Wc, Wa, Cb, Cc, Sb, Sc, Sa);
        if (r + 2 > b1) break;
        iter(r + 2, Wc, Wa, Wb, Cc, Ca, Sc, Sa, Sb);
    }

    smax = wave_max(smax);
    if (lane == 0) slot_add(p.slots[p.s_out], blockIdx.x, smax);
    if (__any(bad) && lane == 0) raise_flag(p.flag);
}

// ---- both stages in one launch, grids of up to a few workgroups per CU ---------------------------
//
// A workgroup of eight wavefronts holds a strip of 56 columns and a segment of up
// to kBlockRows - 4 rows: the wavefronts first form a share each of the segment's
// U* rows (and two more on either side) into LDS, in primitive form, then, after a
// barrier, a share each of the output rows, whose U^n they read again.  In the march
// above every wavefront forms four U* rows of its neighbours' and runs the two stages
// one after the other on one wavefront per SIMD; here that is four rows per eight
// wavefronts, and the eight share the rows of both stages: 100^2 15.5 -> 9.4 us per
// step, 512^2 24.5 -> 18.9, 1000 x 700 33.0 -> 30.8 (FP32 13.3 -> 7.4, 21.4 -> 14.4,
// 26.4 -> 22.2).  Bound by the latency of a wavefront's few rows on small grids; on the
// larger ones FP64 issue takes 18 of 30 us (1000 x 700: 10.1 M wave instructions) and
// the wavefronts wait 31% of their cycles (two on a SIMD, the uneven shares at the
// barrier and the end).  One workgroup on a CU in FP64 (LDS), two in FP32;
// twelve wavefronts measured 5% slower (each adds a face per stage), sixteen spill.
constexpr int kBlockWaves = 8;
constexpr int kBlockCols = 60;  // U* columns kept: lanes 2..61
constexpr int kBlockRows = 56;  // U* rows: 157.5 KB in FP64

// half slopes from the differences below and above
template <typename T>
__device__ __forceinline__ Prim<T> mc_half_diff(const Prim<T>& a, const Prim<T>& b)
{
    return {mc_half(a.r, b.r),     mc_half(a.u, b.u),     mc_half(a.v, b.v),
            mc_half(a.pxx, b.pxx), mc_half(a.pxy, b.pxy), mc_half(a.pyy, b.pyy)};
}

// One stage of a wavefront on the rows [ra, rb) of its columns.  fetch(r): row r of
// U^n; state(r, C): the primitive row r the stage acts on, given that row; rows
// ra - 2 .. rb + 1.  emit(r, U) takes the results.
template <typename T, class Fetch, class State, class Emit>
__device__ __forceinline__ void kt_march(int ra, int rb, T cx, T cy, Fetch fetch, State state, Emit emit)
{
    if (ra >= rb) return;
    Cons<T> Ca = fetch(ra + 1), Cb = fetch(ra - 1), Cc = fetch(ra);
    const Prim<T> below = state(ra - 2, fetch(ra - 2));
    Prim<T> Wa = state(ra + 1, Ca), Wb = state(ra - 1, Cb), Wc = state(ra, Cc);
    Prim<T> high = plus(Wb, mc_half_slope(below, Wb, Wc));  // high y-face state of the row below
    Cons<T> acc{};
    // (W0, C0) row r, Wm and Wp the rows below and above; (Wm, Cm) take row r + 2
    auto row = [&](int r, Prim<T>& Wm, Cons<T>& Cm, const Prim<T>& W0, const Cons<T>& C0, const Prim<T>& Wp) {
        const Cons<T> next = fetch(min(r + 2, rb + 1));  // past the end: a row already read
        const Prim<T> sy = mc_half_slope(Wm, W0, Wp);
        const Cons<T> G = swap(kt_flux2_x(swap(high), swap(sub(W0, sy))));  // face r - 1/2
        if (r > ra)
            emit(r - 1, Cons<T>{acc.r - cy * G.r, acc.mx - cy * G.mx, acc.my - cy * G.my, acc.exx - cy * G.exx,
                                acc.exy - cy * G.exy, acc.eyy - cy * G.eyy});
        if (r < rb) {
            const Prim<T> drx = sub(lane_shift<+1>(W0), W0);
            const Prim<T> sx = mc_half_diff(lane_shift<-1>(drx), drx);
            const Cons<T> F = kt_flux2_x(plus(W0, sx), lane_shift<+1>(sub(W0, sx)));
            const Cons<T> Fm = lane_shift<-1>(F);
            acc = {C0.r - cx * (F.r - Fm.r) + cy * G.r,         C0.mx - cx * (F.mx - Fm.mx) + cy * G.mx,
                   C0.my - cx * (F.my - Fm.my) + cy * G.my,     C0.exx - cx * (F.exx - Fm.exx) + cy * G.exx,
                   C0.exy - cx * (F.exy - Fm.exy) + cy * G.exy, C0.eyy - cx * (F.eyy - Fm.eyy) + cy * G.eyy};
        }
        high = plus(W0, sy);
        Wm = state(min(r + 2, rb + 1), next);
        Cm = next;
    };
    for (int r = ra; r <= rb; r += 3) {
        row(r, Wb, Cb, Wc, Cc, Wa);
        if (r + 1 > rb) break;
        row(r + 1, Wc, Cc, Wa, Ca, Wb);
        if (r + 2 > rb) break;
        row(r + 2, Wa, Ca, Wb, Cb, Wc);
    }
}

template <typename T>
__global__ __launch_bounds__(64 * kBlockWaves, 2) void kt_block_kernel(StepArgs<T> p)
{
    __shared__ T star[kBlockRows][6][kBlockCols];
    double t_now;
    const double dt = kt_dt(p, &t_now);
    if (blockIdx.x == 0) {
        slot_clear(p.slots[p.s_reset], threadIdx.x);
        if (threadIdx.x == 0) {
            p.slots[p.s_out].t = t_now + dt;
            if (p.dt_log) *p.dt_log = dt;
        }
    }
    const int lane = threadIdx.x & 63, w = wave_in_block();
    const unsigned unit = xcd_block(blockIdx.x, gridDim.x);
    const int sx = unit % p.nstrips, sy = unit / p.nstrips;
    const int c0 = sx * kFusedStrip - 4, c = c0 + lane;  // columns of lane 0, of this lane
    const int gc = map_index(c, p.nx, p.bcx);
    const bool own = lane >= 4 && lane < 4 + kFusedStrip && c < p.nx;
    const int y0 = sy * p.ty, y1 = min(y0 + p.ty, p.ny);
    const Planes<T> in(p.U, (size_t)p.nx * p.ny);
    const OutPlanes<T> out(p.Unew, (size_t)p.nx * p.ny);
    auto fetch = [&](int r) -> Cons<T> { return in.load((unsigned)(map_near(map_near(r, p.ny, p.bcy), p.ny, p.bcy) * p.nx + gc)); };
    // rows [a, b) shared out: this wavefront's first row
    auto share = [&](int a, int b, int i) { return a + (b - a) * i / kBlockWaves; };

    const T h1 = T(0.25 * dt / p.dx), h2 = T(0.25 * dt / p.dy);  // half the stage's length, of 2H
    kt_march<T>(
        share(y0 - 2, y1 + 2, w), share(y0 - 2, y1 + 2, w + 1), h1, h2, fetch,
        [](int, const Cons<T>& C) { return to_prim(C); },
        [&](int r, const Cons<T>& U) {
            if (lane < 2 || lane >= 2 + kBlockCols) return;
            T(*const q)[kBlockCols] = star[r - (y0 - 2)];
            const Prim<T> s = to_prim(U);
            q[0][lane - 2] = s.r;
            q[1][lane - 2] = s.u;
            q[2][lane - 2] = s.v;
            q[3][lane - 2] = s.pxx;
            q[4][lane - 2] = s.pxy;
            q[5][lane - 2] = s.pyy;
        });
    __syncthreads();

    // the column of U* this lane reads: its own (a torus window on a periodic axis), the
    // edge column's on outflow; lanes outside 2..61 feed nothing that is used
    const int src = p.bcx != 0 ? min(max(c, 0), p.nx - 1) - c0 : lane;
    const int col = min(max(src - 2, 0), kBlockCols - 1);
    double smax = 0.0;
    bool bad = false;
    const double idx = 1.0 / p.dx, idy = 1.0 / p.dy;
    kt_march<T>(
        share(y0, y1, w), share(y0, y1, w + 1), h1 + h1, h2 + h2, fetch,
        [&](int r, const Cons<T>&) -> Prim<T> {
            const int e = p.bcy != 0 ? min(max(r, 0), p.ny - 1) : r;  // outflow: the edge row
            const T(*const q)[kBlockCols] = star[e - (y0 - 2)];
            return {q[0][col], q[1][col], q[2][col], q[3][col], q[4][col], q[5][col]};
        },
        [&](int r, Cons<T> Un) {
            kick(Un, p, dt, c, r, true);
            if (own) {
                out.store((unsigned)(r * p.nx + c), Un);
                smax = fmax(smax, checked_rate(Un, idx, idy, bad));
            }
        });
    smax = wave_max(smax);
    if (lane == 0) slot_add(p.slots[p.s_out], blockIdx.x, smax);
    if (__any(bad) && lane == 0) raise_flag(p.flag);
}

// Which kernel, and how many rows per segment (at most the grid's): the least of the
// times (ns) below.
//
// March: the critical-path rule of the sweep, with its halo (stage 1 forms six rows
// more than the segment's, stage 2 two, an average of four per row) and rounds of
// 1024 wavefronts.  A row takes 1.74 us (FP32 1.3), the launch 3 (4).
// Block: the longest share of either stage; a round is 256 workgroups (FP32: 512,
// two on a CU, or a single one each).  A row of one stage takes 1.75 us with two
// wavefronts on the SIMD (FP32 1.17, with four 1.5), the launch, the barrier and the
// faces of a share 6.5 (5, 8).
// Measured, march / block, us: FP64 100^2 15.5 / 9.4, 512^2 24.5 / 18.9, 700^2
// 26.5 / 24.6, 1000 x 700 33.0 / 30.8; in more than one round, whose workgroups follow
// one another on a CU, barrier and launch each time, 1024^2 44 / 51.5, 1500^2 80 / 111,
// 100000 x 2 27 / 57, 30000 x 8 24 / 31, 60000 x 20 59 / 74: the march.  FP32 1400^2
// (two rounds) 53 / 46, 2048^2 (three) 104 / 87, 3000^2 (seven) 171 / 195: past three
// rounds the march, whose wavefronts then overlap, is taken.
KtPlan kt_plan(int nx, int ny, bool f64)
{
    const long strips = (nx + kFusedStrip - 1) / kFusedStrip;
    auto segs = [&](int t) { return strips * ((ny + t - 1) / t); };
    KtPlan best{false, 0};
    long best_ns = -1;
    auto offer = [&](bool block, int t, long ns) {
        if (best_ns < 0 || ns < best_ns) {
            best_ns = ns;
            best = {block, t};
        }
    };
    for (int t = std::min(segs(8) >= 256 ? 8 : 4, ny); t <= std::min(96, ny); ++t) {
        const long rows = ((segs(t) + 1023) / 1024) * (t + 4);
        offer(false, t, f64 ? 3000 + 1740 * rows : 4000 + 1300 * rows);
    }
    auto share = [](int n) { return (n + kBlockWaves - 1) / kBlockWaves; };
    for (int t = std::min(kBlockRows - 4, ny); t >= 1; --t) {
        const long n = segs(t), rows = share(t + 4) + share(t);
        if (n <= 256) offer(true, t, f64 ? 6500 + 1750 * rows : 5000 + 1170 * rows);
        else if (!f64 && n <= 3 * 512) offer(true, t, (8000 + 1500 * rows) * ((n + 511) / 512));
    }
    return best;
}

template <typename T>
hipError_t launch_kt_fused(StepArgs<T> a, KtPlan plan, hipStream_t s)
{
    if (const char* e = std::getenv("CSH_KT_ROWS")) {
        const int v = std::atoi(e);
        if (v >= 1) plan = {false, v};
    }
    a.nstrips = (a.nx + kFusedStrip - 1) / kFusedStrip;
    a.ty = plan.rows;
    a.nsegs = (a.ny + a.ty - 1) / a.ty;
    if (plan.block) {
        kt_block_kernel<T><<<dim3(a.nstrips * a.nsegs), dim3(64 * kBlockWaves), 0, s>>>(a);
        return hipGetLastError();
    }
    const int nwaves = a.nstrips * a.nsegs;
    kt_fused_kernel<T><<<dim3((nwaves + kWaves - 1) / kWaves), dim3(64 * kWaves), 0, s>>>(a);
    return hipGetLastError();
}

template hipError_t launch_kt_fused<double>(StepArgs<double>, KtPlan, hipStream_t);
template hipError_t launch_kt_fused<float>(StepArgs<float>, KtPlan, hipStream_t);

template <typename T>
hipError_t launch_kt(const StepArgs<T>& a, bool final_stage, hipStream_t s)
{
    const dim3 grid((a.nstrips + kWaves - 1) / kWaves), block(64 * kWaves);
    if (final_stage) kt_kernel<T, true><<<grid, block, 0, s>>>(a);
    else kt_kernel<T, false><<<grid, block, 0, s>>>(a);
    return hipGetLastError();
}

template hipError_t launch_kt<double>(const StepArgs<double>&, bool, hipStream_t);
template hipError_t launch_kt<float>(const StepArgs<float>&, bool, hipStream_t);

}  // namespace csh
