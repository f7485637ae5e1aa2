// Forward sweep kernels of the collisionless-stellar-hydrodynamics scheme
// (Mitchell, Vorobyov & Hensler, arXiv:1210.5246, Sec. 3.3), gfx950.
//
// One sweep = MUSCL-Hancock with characteristic tracing (eqs. (19)-(32)), an
// HLL flux at every face, the dimensionally unsplit conservative update, the
// operator-split external-gravity kick (Sec. 3.3, last paragraph) and the
// fused reduction of the CFL rate of the new state.
//
// Work decomposition (2-D): one wavefront owns a strip of 60 output columns
// and marches up a segment of rows.  Lane l holds column x0 - 2 + l, so the
// two lanes at each edge are the stencil halo.  x neighbours come from lane
// shuffles; the rows r-1, r, r+1 the y slopes need, the flux of the previous
// row and the high y-face state of the cell below stay in registers.  No
// second pass: each input cell is read from HBM once per strip it belongs to
// (64/60 columns) and each output cell is written once.  LDS carries only the
// faces between the rows of two wavefronts (small grids).
#include <type_traits>

#include "csh_device.h"
#include "csh_internal.h"
#include "csh_xcd.h"

namespace csh {

template <typename T>
__device__ __forceinline__ double step_dt(const StepArgs<T>& p, double* t_now)
{
    const Slot& sl = p.slots[p.s_in];
    const double t = sl.t;
    *t_now = t;
    if (!p.dev_dt) return p.dt_in ? *p.dt_in : p.dt;
    double dt = p.cfl / slot_rate(sl);
    if (p.t_end > 0.0) {
        if (t >= p.t_end) dt = 0.0;
        else if (t + dt > p.t_end) dt = p.t_end - t;
    }
    return dt;
}

// The step's time and log, and the slot of the step after cleared (one workgroup).
template <typename T>
__device__ __forceinline__ void open_step(const StepArgs<T>& p, double t_now, double dt)
{
    if (blockIdx.x != 0) return;
    slot_clear(p.slots[p.s_reset], threadIdx.x);
    if (threadIdx.x == 0) {
        p.slots[p.s_out].t = t_now + dt;
        if (p.dt_log) *p.dt_log = dt;
    }
}

// The wavefront's CFL rate into the output slot, and the non-physical flag.
template <typename T>
__device__ __forceinline__ void close_step(const StepArgs<T>& p, int lane, double smax, bool bad)
{
    smax = wave_max(smax);
    if (lane == 0) slot_add(p.slots[p.s_out], blockIdx.x, smax);
    if (__any(bad) && lane == 0) raise_flag(p.flag);
}

// One-dimensional grids: a lane per cell, 60 cells per wavefront (two halo
// lanes per side).
template <typename T, bool FLUXES, int RS>
__global__ __launch_bounds__(64 * kWaves) void sweep1d_kernel(StepArgs<T> p)
{
    double t_now;
    const double dt = step_dt(p, &t_now);
    if (!FLUXES) open_step(p, t_now, dt);
    const int lane = threadIdx.x & 63;
    const int wid = blockIdx.x * kWaves + wave_in_block();
    if (wid >= p.nstrips) return;  // uniform per wavefront
    const int c = wid * kStrip - 2 + lane;  // cell of this lane
    const Cons<T> U0 = load_cons(p.U, (size_t)p.nx, (size_t)map_index(c, p.nx, p.bcx));
    const Cons<T> F = flux_1d<T, RS>(U0, T(dt / (2.0 * p.dx)));  // face c + 1/2
    if constexpr (FLUXES) {
        // lanes 1..61 hold faces x0 - 1/2 .. x0 + 59 + 1/2
        if (lane >= 1 && lane <= 1 + kStrip && c >= -1 && c <= p.nx - 1)
            store_cons(p.Fx, (size_t)(p.nx + 1), (size_t)(c + 1), F);
        return;
    }
    double smax = 0.0;
    bool bad = false;
    Cons<T> Un = update(U0, T(dt / p.dx), F, lane_shift<-1>(F));
    kick(Un, p, dt, c, 0, false);
    if (lane >= 2 && lane < 2 + kStrip && c < p.nx) {
        store_cons(p.Unew, (size_t)p.nx, (size_t)c, Un);
        smax = checked_rate<T, false>(Un, 1.0 / p.dx, 0.0, bad);
    }
    close_step(p, lane, smax, bad);
}

// Two-dimensional grids.  A row's work: the face states of its cells, the y flux
// at their low faces (against the high states of the row below, in registers),
// which finishes the row below, and the x fluxes.  A wavefront marches its rows
// from the bottom up.
//
// STACKED: the four wavefronts of a workgroup hold the rows y0 - 1 .. y1 of one
// strip (rows y0 .. y1 - 1 are the outputs), a quarter each.  At the face between
// two wavefronts' rows the lower one publishes its last high states when its
// march ends; the upper one then forms the flux from its first low states,
// finishes its first row and publishes the flux, with which the lower one
// finishes its last row.  So two rows per workgroup are traced twice, not two per
// wavefront: a small grid leaves a few rows to each wavefront, and with one
// wavefront per SIMD a row takes ~2900 cycles (2280 of them issue).
// Else each wavefront has a segment of its own, as many independent wavefronts
// as fit: for grids with many rows per SIMD, bound by FP64 issue (VALU busy 0.86
// at 4096^2, 0.42-0.43 ms per step).  The stacked workgroups are numbered XCD-aware:
// neighbouring strips share the 128-byte lines at their edges, in reads and in
// partial writes, and so meet in one L2 (us per step in the hardware's order / so:
// FP64 300 x 200 8.6 / 7.7, 512^2 15.0 / 14.0, 700 x 500 16.6 / 16.0; FP32 2048^2
// 62.7 / 60.4, 4096^2 259 / 237).
template <typename T, bool FLUXES, int RS, bool STACKED>
__global__ __launch_bounds__(64 * kWaves) void sweep_kernel(StepArgs<T> p)
{
    // per wavefront: of its first row the low y-face state, the update without
    // its y fluxes and the flux at its high face (read by the same lane only);
    // the high y-face state of its last row (for the wavefront above) and the
    // flux at the low face of its first row (for the one below)
    enum { kLow, kFirst, kFirstHigh, kHigh, kFlux, kSlots };
    __shared__ T xch[STACKED ? kWaves : 1][kSlots][6][64];
    double t_now;
    const double dt = step_dt(p, &t_now);
    if (!FLUXES) open_step(p, t_now, dt);

    const int lane = threadIdx.x & 63, w = wave_in_block();
    // STACKED: the workgroup's wavefronts share one strip and segment; else each
    // wavefront has its own
    unsigned unit = xcd_block(blockIdx.x, gridDim.x);
    if constexpr (!STACKED) {
        unit = blockIdx.x * kWaves + w;
        if (unit >= (unsigned)(p.nstrips * p.nsegs)) return;  // uniform per wavefront
    }
    const int sx = unit % p.nstrips, sy = unit / p.nstrips;
    const int c = sx * kStrip - 2 + lane;  // column of this lane
    const int gc = map_index(c, p.nx, p.bcx);
    const bool own = lane >= 2 && lane < 2 + kStrip && c < p.nx;  // lane owns an output column
    const size_t plane = (size_t)p.nx * p.ny;
    const int y0 = sy * p.ty, y1 = min(y0 + p.ty, p.ny);
    // rows [ra, rb) of this wavefront
    const int ra = STACKED ? y0 - 1 + w * p.tw : y0 - 1, rb = STACKED ? min(ra + p.tw, y1 + 1) : y1 + 1;
    const bool any = !STACKED || ra < rb;

    const T kx = T(dt / (2.0 * p.dx)), cx = T(dt / p.dx), ky = T(dt / (2.0 * p.dy)), cy = T(dt / p.dy);
    const double idx = 1.0 / p.dx, idy = 1.0 / p.dy;
    double smax = 0.0;
    bool bad = false;
    const Planes<T> in(p.U, plane);
    const OutPlanes<T> out(p.Unew, plane);
    auto put = [&](int slot, const T (&v)[6]) {
#pragma unroll
        for (int k = 0; k < 6; ++k) xch[w][slot][k][lane] = v[k];
    };
    auto put_p = [&](int slot, const Prim<T>& v) { put(slot, {v.r, v.u, v.v, v.pxx, v.pxy, v.pyy}); };
    auto put_c = [&](int slot, const Cons<T>& v) { put(slot, {v.r, v.mx, v.my, v.exx, v.exy, v.eyy}); };
    auto get_p = [&](int wave, int slot) -> Prim<T> {
        const T(*q)[64] = xch[wave][slot];
        return {q[0][lane], q[1][lane], q[2][lane], q[3][lane], q[4][lane], q[5][lane]};
    };
    auto get_c = [&](int wave, int slot) -> Cons<T> {
        const T(*q)[64] = xch[wave][slot];
        return {q[0][lane], q[1][lane], q[2][lane], q[3][lane], q[4][lane], q[5][lane]};
    };
    // y flux between the high state of the cell below and the low state of the cell above
    auto y_flux = [&](const Prim<T>& below, const Prim<T>& above) -> Cons<T> {
        return swap(riemann_x<RS>(make_face_x(swap(below)), make_face_x(swap(above))));
    };
    auto plus_cy = [&](const Cons<T>& a, T s, const Cons<T>& G) -> Cons<T> {
        return {a.r + s * G.r,     a.mx + s * G.mx,   a.my + s * G.my,
                a.exx + s * G.exx, a.exy + s * G.exy, a.eyy + s * G.eyy};
    };
    // cell (c, r) from its update without and the flux through its high y face
    auto finish = [&](int r, const Cons<T>& a, const Cons<T>& G) {
        Cons<T> Un = plus_cy(a, -cy, G);
        kick(Un, p, dt, c, r, true);
        if (own) {
            out.store((unsigned)(r * p.nx + c), Un);
            smax = fmax(smax, checked_rate(Un, idx, idy, bad));
        }
    };

    Cons<T> acc{};  // update of the cell below, all but its high y-face flux
    Prim<T> yhi_prev{};  // high y-face state of the cell below (primitive, axes not exchanged)
    if (any) {
        auto load_row = [&](int r) -> Cons<T> {
            const int gr = map_near(r, p.ny, p.bcy);  // rows ra - 1 .. rb, ny >= 2
            return in.load((unsigned)(gr * p.nx + gc));
        };
        // Row window in three rotating register sets: the set holding row r-1
        // is refilled with row r+2, so the window advances without moves.
        Cons<T> Ua = load_row(ra - 1), Ub = load_row(ra), Uc = load_row(ra + 1);
        T ia = rcp(Ua.r), ib = rcp(Ub.r), ic = rcp(Uc.r);
        Prim<T> Wa = to_prim(Ua, ia), Wb = to_prim(Ub, ib), Wc = to_prim(Uc, ic);
        Prim<T> dly = sub(Wb, Wa);  // y difference below the row: the previous row's upper one

        // one row: (Um, Wm) row r-1 (refilled with row r+2), (U0, W0, ir0) row r, Wp row r+1;
        // first: row ra, whose low y flux is not formed here
        auto row = [&](auto first, int r, Cons<T>& Um, Prim<T>& Wm, T& irm, const Cons<T>& U0, const Prim<T>& W0,
                       T ir0, const Prim<T>& Wp) {
            const Cons<T> Unext = load_row(min(r + 2, rb));  // past the window's end: a row already read

            // face states of (c, r): the x differences from the right neighbour (a lane
            // shift), the left one that of the lane to the left; the y difference below
            // the row carried from the row before
            const Prim<T> drx = sub(lane_shift<+1>(W0), W0), dry = sub(Wp, W0);
            const Faces<T> fs = face_states_d<T, true>(W0, ir0, lane_shift<-1>(drx), drx, dly, dry, kx, ky);
            dly = dry;

            // x faces of row r: fluxes out, or the update of (c, r) without its y fluxes
            auto x_part = [&]() -> Cons<T> {
                const Cons<T> F = riemann_x<RS>(make_face_x(fs.xhi), make_face_x(lane_shift<+1>(fs.xlo)));
                if constexpr (FLUXES) {
                    if (lane >= 1 && lane <= 1 + kStrip && c >= -1 && c <= p.nx - 1)
                        store_cons(p.Fx, (size_t)(p.nx + 1) * p.ny, (size_t)r * (p.nx + 1) + (c + 1), F);
                    return F;
                } else {
                    return update(U0, cx, F, lane_shift<-1>(F));
                }
            };
            if constexpr (first.value) {
                if constexpr (STACKED) {
                    put_p(kLow, fs.ylo);
                    if (w > 0 && r < y1) acc = x_part();
                }
            } else {
                const Cons<T> G = y_flux(yhi_prev, fs.ylo);  // y face r - 1/2
                if constexpr (FLUXES) {
                    if (own) store_cons(p.Fy, (size_t)p.nx * (p.ny + 1), (size_t)r * p.nx + c, G);
                } else if (r - 1 > ra) {
                    finish(r - 1, acc, G);
                } else if (STACKED && w > 0) {  // the wavefront's first row: its low flux comes last
                    put_c(kFirst, acc);
                    put_c(kFirstHigh, G);
                }
                // the update of (c, r) with its x fluxes and its low y flux
                if (r < y1) acc = plus_cy(x_part(), cy, G);
            }
            yhi_prev = fs.yhi;
            Um = Unext;  // row r + 2 takes the place of row r - 1
            irm = rcp(Unext.r);
            Wm = to_prim(Unext, irm);
        };
        constexpr std::true_type first{};
        constexpr std::false_type later{};

        row(first, ra, Ua, Wa, ia, Ub, Wb, ib, Wc);
        for (int r = ra + 1; r < rb; r += 3) {
            row(later, r, Ub, Wb, ib, Uc, Wc, ic, Wa);
            if (r + 1 >= rb) break;
            row(later, r + 1, Uc, Wc, ic, Ua, Wa, ia, Wb);
            if (r + 2 >= rb) break;
            row(later, r + 2, Ua, Wa, ia, Ub, Wb, ib, Wc);
        }
        if constexpr (STACKED) put_p(kHigh, yhi_prev);
    }

    if constexpr (STACKED) {
        // the faces between the wavefronts' rows (wavefront w - 1's rows end where w's begin)
        __syncthreads();
        if (any && w > 0) {
            const Cons<T> G = y_flux(get_p(w - 1, kHigh), get_p(w, kLow));
            if constexpr (FLUXES) {
                if (own) store_cons(p.Fy, (size_t)p.nx * (p.ny + 1), (size_t)ra * p.nx + c, G);
            } else {
                put_c(kFlux, G);
                if (rb - ra == 1) acc = plus_cy(acc, cy, G);
                else finish(ra, plus_cy(get_c(w, kFirst), cy, G), get_c(w, kFirstHigh));
            }
        }
        if constexpr (!FLUXES) {
            __syncthreads();
            // the last row, unless it lies outside the outputs (then the march finished the one below it)
            if (any && rb - 1 >= y0 && rb - 1 < y1) finish(rb - 1, acc, get_c(w + 1, kFlux));
        }
    }
    if constexpr (!FLUXES) close_step(p, lane, smax, bad);
}

template <typename T, bool FLUXES, int RS>
void launch_sweep(const StepArgs<T>& a, bool twod, hipStream_t s)
{
    const dim3 block(64 * kWaves);
    const unsigned units = (unsigned)(a.nstrips * a.nsegs);
    if (!twod) sweep1d_kernel<T, FLUXES, RS><<<(a.nstrips + kWaves - 1) / kWaves, block, 0, s>>>(a);
    else if (sizeof(T) == 4 || a.tw > 0) sweep_kernel<T, FLUXES, RS, true><<<units, block, 0, s>>>(a);
    else if constexpr (sizeof(T) == 8)
        sweep_kernel<T, FLUXES, RS, false><<<(units + kWaves - 1) / kWaves, block, 0, s>>>(a);
}

template <typename T>
hipError_t launch_step(const StepArgs<T>& a, bool twod, bool fluxes, int solver, hipStream_t s)
{
    if (solver == 1) {
        if (fluxes) launch_sweep<T, true, 1>(a, twod, s);
        else launch_sweep<T, false, 1>(a, twod, s);
    } else {
        if (fluxes) launch_sweep<T, true, 0>(a, twod, s);
        else launch_sweep<T, false, 0>(a, twod, s);
    }
    return hipGetLastError();
}

// ---- primitive -> conserved, with validation ------------------------------------------------

template <typename T>
__global__ __launch_bounds__(256) void init_kernel(const T* __restrict__ W, T* __restrict__ U, int64_t n,
                                                   int* flag)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = false;
    if (c < n) {
        const Prim<T> w = {W[c], W[n + c], W[2 * n + c], W[3 * n + c], W[4 * n + c], W[5 * n + c]};
        bad = !physical(w);
        store_cons(U, (size_t)n, (size_t)c, to_cons(w));
    }
    if (__any(bad) && (threadIdx.x & 63) == 0) raise_flag(flag);
}

template <typename T>
hipError_t launch_init(const T* W, T* U, int64_t n, int* flag, hipStream_t s)
{
    const int64_t blocks = (n + 255) / 256;
    init_kernel<T><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(W, U, n, flag);
    return hipGetLastError();
}

// ---- standalone CFL-rate reduction ----------------------------------------------------------------

// Two cells per thread and iteration (their loads issued together), a
// workgroup maximum in LDS and one 64-bit atomic per workgroup.
template <typename T>
__global__ __launch_bounds__(256) void maxspeed_kernel(const T* __restrict__ U, int64_t n, int twod,
                                                       double idx, double idy, Slot* slot, int* flag)
{
    double s = 0.0;
    bool bad = false;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += 2 * stride) {
        const int64_t c2 = c + stride;
        const Cons<T> ua = load_cons(U, (size_t)n, (size_t)c);
        const Cons<T> ub = load_cons(U, (size_t)n, (size_t)(c2 < n ? c2 : c));
        const Prim<T> wa = to_prim(ua), wb = to_prim(ub);
        s = fmax(s, twod ? signal_rate<T, true>(wa, idx, idy) : signal_rate<T, false>(wa, idx, idy));
        s = fmax(s, twod ? signal_rate<T, true>(wb, idx, idy) : signal_rate<T, false>(wb, idx, idy));
        bad = bad || !physical(wa) || !physical(wb);
    }
    s = wave_max(s);
    __shared__ double red[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) red[wv] = s;
    if (__any(bad) && lane == 0) raise_flag(flag);
    __syncthreads();
    if (threadIdx.x == 0) slot_add(*slot, blockIdx.x, fmax(fmax(red[0], red[1]), fmax(red[2], red[3])));
}

template <typename T>
hipError_t launch_maxspeed(const T* U, int nx, int ny, double dx, double dy, Slot* slot, int* flag,
                           hipStream_t s)
{
    const int64_t n = (int64_t)nx * ny;
    int64_t blocks = (n + 511) / 512;
    if (blocks > 4096) blocks = 4096;
    maxspeed_kernel<T><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(U, n, ny > 1, 1.0 / dx,
                                                                    ny > 1 ? 1.0 / dy : 0.0, slot, flag);
    return hipGetLastError();
}

__global__ void reset_kernel(Slot* slots, int nslots, double t0)
{
    for (int i = 0; i < nslots; ++i) slot_clear(slots[i], threadIdx.x);
    if ((int)threadIdx.x < nslots) slots[threadIdx.x].t = t0;
}

hipError_t launch_reset(Slot* slots, int nslots, double t0, hipStream_t s)
{
    reset_kernel<<<1, 64, 0, s>>>(slots, nslots, t0);
    return hipGetLastError();
}

__global__ void publish_kernel(const Slot* slot, HostCell* cell)
{
    const double s = slot_rate(*slot);
    if (threadIdx.x == 0) cell->rate = s;
}

hipError_t launch_publish(const Slot* slot, HostCell* cell, hipStream_t s)
{
    publish_kernel<<<1, 64, 0, s>>>(slot, cell);
    return hipGetLastError();
}

__global__ void clear_flag_kernel(int* flag) { *flag = 0; }

hipError_t launch_clear_flag(int* flag, hipStream_t s)
{
    clear_flag_kernel<<<1, 1, 0, s>>>(flag);
    return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(256) void copy_kernel(const T* __restrict__ a, T* __restrict__ b, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        b[i] = a[i];
}

template <typename T>
hipError_t launch_copy(const T* src, T* dst, int64_t n, hipStream_t s)
{
    int64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    copy_kernel<T><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(src, dst, n);
    return hipGetLastError();
}

#define CSH_INSTANTIATE(T)                                                                         \
    template hipError_t launch_step<T>(const StepArgs<T>&, bool, bool, int, hipStream_t);               \
    template hipError_t launch_init<T>(const T*, T*, int64_t, int*, hipStream_t);                  \
    template hipError_t launch_maxspeed<T>(const T*, int, int, double, double, Slot*, int*,        \
                                           hipStream_t);                                           \
    template hipError_t launch_copy<T>(const T*, T*, int64_t, hipStream_t);

CSH_INSTANTIATE(double)
CSH_INSTANTIATE(float)

}  // namespace csh
