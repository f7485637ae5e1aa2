// Whole runs of a short 1-D grid in one launch (gfx950).
//
// A 1-D grid of at most kLineCells cells fits one workgroup: a lane per cell,
// 60 cells per wavefront as in the 1-D sweep.  The workgroup takes all steps of
// csh_run_cfl, csh_run_dts or csh_run_cfl_states itself: each step the
// wavefronts publish their new cells in LDS, one barrier, every lane reads its
// cell (the halo lanes their neighbours' or boundary cells), and every thread
// forms the next timestep from the wavefronts' CFL maxima.  A launch per step
// is bound by the launch and by the reduction through memory (256 cells: 3.3 us per
// step in a replayed graph, 4.5 launched one by one); here a step is the serial chain
// of one cell-update, an LDS exchange and a barrier (1.0 us at 60 cells, 1.3 at 240,
// 1.7 at 256, where the fifth wavefront shares a SIMD, 3.2 at 960).  Above kLineCells
// a workgroup would need more wavefronts than a CU holds.
#include "csh_device.h"
#include "csh_internal.h"

namespace csh {

namespace {

constexpr int kMaxWaves = 16;

// twice the Kurganov-Tadmor flux through the high face of the lane's cell
template <typename T>
__device__ __forceinline__ Cons<T> kt_flux2_1d(const Cons<T>& U)
{
    const Prim<T> W = to_prim(U);
    const Prim<T> s = mc_half_slope(lane_shift<-1>(W), W, lane_shift<+1>(W));
    return kt_flux2_x(plus(W, s), lane_shift<+1>(sub(W, s)));
}

// SCHEME: 0 characteristic with HLL, 1 with HLLC, 2 Kurganov-Tadmor
template <typename T, int SCHEME>
__global__ __launch_bounds__(64 * kMaxWaves) void line_run_kernel(LineArgs<T> p)
{
    __shared__ T state[2][6][kLineCells];
    __shared__ double red[2][kMaxWaves];
    const int lane = threadIdx.x & 63, w = wave_in_block(), nw = blockDim.x >> 6;
    const int c = w * kStrip - 2 + lane;
    const int gc = map_index(c, p.nx, p.bcx);
    const bool own = lane >= 2 && lane < 2 + kStrip && c < p.nx;
    const double idx = 1.0 / p.dx;
    bool bad = false;

    // the wavefronts' maxima combined (row: one of two used alternately, so that a
    // row is rewritten only after the barrier in between); its barrier also
    // separates the cells written before it from those read after it
    auto block_rate = [&](double s, int row) -> double {
        s = wave_max(s);
        if (lane == 0) red[row][w] = s;
        __syncthreads();
        double m = red[row][0];
        for (int k = 1; k < nw; ++k) m = fmax(m, red[row][k]);
        return m;
    };
    auto put = [&](int b, const Cons<T>& U) {
        state[b][0][c] = U.r;
        state[b][1][c] = U.mx;
        state[b][2][c] = U.my;
        state[b][3][c] = U.exx;
        state[b][4][c] = U.exy;
        state[b][5][c] = U.eyy;
    };
    auto get = [&](int b) -> Cons<T> {
        return {state[b][0][gc], state[b][1][gc], state[b][2][gc],
                state[b][3][gc], state[b][4][gc], state[b][5][gc]};
    };
    auto rate = [&](const Cons<T>& U) -> double {
        bool b = false;
        const double s = checked_rate<T, false>(U, idx, 0.0, b);
        bad |= own && b;
        return own ? s : 0.0;
    };

    Cons<T> U = load_cons(p.U0, (size_t)p.nx, (size_t)gc);
    double s = block_rate(rate(U), 0), t = 0.0;
    double dt_next = p.dts ? p.dts[0] : 0.0;
    for (int k = 0; k < p.nsteps; ++k) {
        double dt = dt_next;
        if (p.dts) {
            dt_next = p.dts[min(k + 1, p.nsteps - 1)];
        } else {
            dt = p.cfl / s;
            if (p.t_end > 0.0) {
                if (t >= p.t_end) {  // done: the remaining steps leave the state as it is
                    if (p.dt_log)
                        for (int i = k + (int)threadIdx.x; i < p.nsteps; i += blockDim.x) p.dt_log[i] = 0.0;
                    break;
                }
                if (t + dt > p.t_end) dt = p.t_end - t;
            }
        }
        if (threadIdx.x == 0 && p.dt_log) p.dt_log[k] = dt;
        t += dt;
        const int b = SCHEME == 2 ? 0 : k & 1;
        // rounded as a single step's factors dt / dx and dt / (2 dx) (halving is exact), not as
        // dt * idx: csh_step repeats a run's states bit for bit, as the reverse pass does
        const double q = div_by(dt, p.dx, idx);
        Cons<T> Un;
        if constexpr (SCHEME == 2) {
            // the midpoint state through buffer 1, then the full step (coefficients: the fluxes are 2H)
            Cons<T> F = kt_flux2_1d(U);
            const Cons<T> Us = update(U, T(0.25 * q), F, lane_shift<-1>(F));
            if (own) put(1, Us);
            __syncthreads();
            F = kt_flux2_1d(get(1));
            Un = update(U, T(0.5 * q), F, lane_shift<-1>(F));
        } else {
            const Cons<T> F = flux_1d<T, SCHEME>(U, T(0.5 * q));
            Un = update(U, T(q), F, lane_shift<-1>(F));
        }
        kick(Un, p, dt, c, 0, false);
        if (own) {
            put(b, Un);
            if (p.states) store_cons(p.states + (size_t)k * 6 * p.nx, (size_t)p.nx, (size_t)c, Un);
        }
        s = block_rate(rate(Un), (k + 1) & 1);
        U = get(b);
    }
    if (own && p.U) store_cons(p.U, (size_t)p.nx, (size_t)c, U);

    // the slots as after the run's last step: rate and time in s_out, the others clear
    for (int i = 0; i < 3; ++i) slot_clear(p.slots[i], threadIdx.x);
    __syncthreads();
    if (threadIdx.x == 0) {
        p.slots[p.s_out].t = t;
        p.slots[p.s_out].part[0].bits = (unsigned long long)__double_as_longlong(s);
    }
    if (__any(bad) && lane == 0) raise_flag(p.flag);
}

}  // namespace

template <typename T>
hipError_t launch_line_run(const LineArgs<T>& a, int scheme, hipStream_t s)
{
    if (a.nx > kLineCells) return hipErrorInvalidValue;
    const int threads = 64 * ((a.nx + kStrip - 1) / kStrip);
    if (scheme == 2) line_run_kernel<T, 2><<<1, threads, 0, s>>>(a);
    else if (scheme == 1) line_run_kernel<T, 1><<<1, threads, 0, s>>>(a);
    else line_run_kernel<T, 0><<<1, threads, 0, s>>>(a);
    return hipGetLastError();
}

template hipError_t launch_line_run<double>(const LineArgs<double>&, int, hipStream_t);
template hipError_t launch_line_run<float>(const LineArgs<float>&, int, hipStream_t);

}  // namespace csh
