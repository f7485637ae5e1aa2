// C ABI of the sweep (declarations and contracts in include/cshydro.h).
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <string>

#include "cshydro.h"
#include "csh_api_util.h"
#include "csh_internal.h"
#include "csh_diag.h"

using csh::Slot;

thread_local std::string csh_err_msg;

extern "C" const char* csh_last_error(void) { return csh_err_msg.c_str(); }

struct csh_grid {
    int nx = 0, ny = 0, bcx = 0, bcy = 0, dtype = CSH_F64;
    double dx = 1, dy = 1;
    double vc = 0, rc = 0, x0 = 0, y0 = 0;
    hipStream_t stream = nullptr;
    hipStream_t capture = nullptr;  // private stream used only to record graphs
    Slot* slots = nullptr;          // 3 device slots (see csh_internal.h)
    csh::HostCell* cell = nullptr;  // pinned: rate and non-physical flag for the host
    int phase = 0;                  // slot holding the rate of the latest output
    int ty = 32;                    // rows per segment of the 2-D sweep
    int tw = 0;                     // rows per wavefront of a stacked segment (0: a wavefront per segment)
    double* adj_ws = nullptr;       // adjoint workspace, allocated on first use
    size_t adj_ws_n = 0;
    int scheme = CSH_SCHEME_MUSCL_HLL;
    csh::KtPlan kt_plan{};          // work decomposition of the 2-D Kurganov-Tadmor step
    void* kt_buf = nullptr;         // stage state of the 1-D Kurganov-Tadmor scheme
    double* fourier_ws = nullptr;   // partial sums + amplitudes of csh_fourier_amplitudes
    // cached graph of csh_run_cfl / csh_run_dts
    hipGraphExec_t exec = nullptr;
    int g_mode = -1, g_nsteps = -1;
    double g_cfl = 0, g_tend = 0;
    const void *g_U = nullptr, *g_W = nullptr, *g_log = nullptr;
    double* log = nullptr;          // the recorded run's timestep log, copied to the caller's
    int log_n = 0;
};

namespace {

// Work decomposition of the 2-D sweep: ty rows per segment and, for a stacked
// segment (a workgroup of kWaves wavefronts on one strip), tw rows per
// wavefront; tw = 0: a wavefront per segment.
//
// Stacked segments trace two halo rows per workgroup instead of two per
// wavefront, at the price of two barriers and a flux exchange at their end
// (about 0.7 of a row).  In FP64 that pays while a launch has few rows per SIMD
// (us per step, stacked / a wavefront per segment: 64^2 5.5 / 10.3, 131 x 93
// 6.1 / 10.5, 300 x 200 8.3 / 12.0, 512^2 13.9 / 17.0, 700 x 500 16.1 / 17.6,
// 800^2 23.4 / 23.0, 1024^2 35.7 / 35.0): the line lies at 8 strip rows per
// SIMD.  Not on wide grids of few rows, whose strips alone are more than the two
// workgroups a CU holds: there most of a workgroup's rows are halo (60000 x 2 13.6 /
// 9.6, 120000 x 3 28.6 / 16.6, 54000 x 8 21.5 / 18.2, their fluxes 10.1 / 8.4, 22.2 /
// 15.8, 19.5 / 17.0; 30000 x 2 8.1 / 8.2, 36000 x 10 17.9 / 19.5).  In FP32, whose rows are too short for the latency of one or two
// wavefronts per SIMD, always (2048^2 66 / 86, 4096^2 240 / 242).
void split_rows(csh_grid* h)
{
    const long strips = (h->nx + csh::kStrip - 1) / csh::kStrip, ny = h->ny;
    const bool thin = strips > 2 * 256 && ny <= 8;
    const bool stacked = h->dtype == CSH_F32 || (strips * ny <= 8L * 1024 && !thin);
    int rows = 0;
    if (const char* e = std::getenv("CSH_ROWS")) rows = std::max(0, std::atoi(e));
    long best_cost = -1;
    if (stacked && rows == 0) {
        // tw rows on each of the wavefronts of a CU, one workgroup after the
        // other; a second resident workgroup fills the first one's stalls
        // (measured 0.88 of twice the time)
        for (int t = 1; t <= 64; ++t) {
            const long per_cu = (strips * ((ny + csh::kWaves * t - 3) / (csh::kWaves * t - 2)) + 255) / 256;
            const long cost = per_cu * (10 * t + 7) * (per_cu > 1 ? 22 : 25);
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                rows = csh::kWaves * t - 2;
            }
        }
    } else if (rows == 0) {
        // The segment length that minimises the critical path of the busiest SIMD:
        // ceil(wavefronts / 1024 SIMDs) wavefronts in turn, each marching its rows
        // plus the two halo rows it re-traces.
        for (int t = 8; t <= 96; ++t) {
            const long cost = ((strips * ((ny + t - 1) / t) + 1023) / 1024) * (t + 2);
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                rows = t;
            }
        }
    }
    rows = (int)std::min<long>(rows, ny);
    h->ty = rows;
    h->tw = stacked ? (rows + 2 + csh::kWaves - 1) / csh::kWaves : 0;
}

// Riemann solver of the characteristic sweep
int solver_of(const csh_grid* h)
{
    return h->scheme == CSH_SCHEME_MUSCL_HLLC ? 1 : 0;
}

template <typename T>
csh::StepArgs<T> base_args(const csh_grid* h)
{
    csh::StepArgs<T> a{};
    a.nx = h->nx;
    a.ny = h->ny;
    a.bcx = h->bcx;
    a.bcy = h->bcy;
    a.dx = h->dx;
    a.dy = h->dy;
    a.nstrips = (h->nx + csh::kStrip - 1) / csh::kStrip;
    a.ty = h->ny > 1 ? h->ty : 1;
    a.tw = h->tw;
    a.nsegs = (h->ny + a.ty - 1) / a.ty;
    a.slots = h->slots;
    a.vc2 = h->vc * h->vc;
    a.rc2 = h->rc * h->rc;
    a.x0 = h->x0;
    a.y0 = h->y0;
    a.flag = &h->cell->flag;
    return a;
}

template <typename T>
hipError_t enqueue_step(csh_grid* h, const void* U, void* Un, int dev_dt, double dt, double cfl,
                        double t_end, double* dt_log, hipStream_t s, const double* dt_in = nullptr)
{
    auto a = base_args<T>(h);
    a.U = static_cast<const T*>(U);
    a.Unew = static_cast<T*>(Un);
    a.dev_dt = dev_dt;
    a.dt = dt;
    a.dt_in = dt_in;
    a.cfl = cfl;
    a.t_end = t_end;
    a.dt_log = dt_log;
    a.s_in = h->phase;
    a.s_out = (h->phase + 1) % 3;
    a.s_reset = (h->phase + 2) % 3;
    if (h->scheme == CSH_SCHEME_KT && h->ny > 1) {
        h->phase = a.s_out;
        return csh::launch_kt_fused<T>(a, h->kt_plan, s);
    }
    if (h->scheme == CSH_SCHEME_KT) {
        // 1-D: stage 1: U -> stage buffer over dt/2; records dt in slot s_in
        auto a1 = a;
        a1.Unew = static_cast<T*>(h->kt_buf);
        a1.dt_log = nullptr;
        hipError_t e = csh::launch_kt<T>(a1, false, s);
        if (e != hipSuccess) return e;
        // stage 2: fluxes of the stage state, update from U over dt
        a.U = static_cast<const T*>(h->kt_buf);
        a.Ubase = static_cast<const T*>(U);
        if (dev_dt) {
            a.dev_dt = 0;
            a.dt_in = &h->slots[h->phase].dt;
        }
        h->phase = a.s_out;
        return csh::launch_kt<T>(a, true, s);
    }
    h->phase = a.s_out;
    return csh::launch_step<T>(a, h->ny > 1, false, solver_of(h), s);
}

hipError_t enqueue_maxspeed(csh_grid* h, const void* U, hipStream_t s)
{
    hipError_t e = csh::launch_reset(h->slots, 3, 0.0, s);
    if (e != hipSuccess) return e;
    if (h->dtype == CSH_F64)
        return csh::launch_maxspeed<double>(static_cast<const double*>(U), h->nx, h->ny, h->dx, h->dy,
                                            h->slots + h->phase, &h->cell->flag, s);
    return csh::launch_maxspeed<float>(static_cast<const float*>(U), h->nx, h->ny, h->dx, h->dy,
                                       h->slots + h->phase, &h->cell->flag, s);
}

int read_rate(csh_grid* h, double* s)
{
    CSH_HIP(csh::launch_publish(h->slots + h->phase, h->cell, h->stream));
    CSH_HIP(hipStreamSynchronize(h->stream));
    *s = h->cell->rate;
    if (h->cell->flag) return csh_fail(CSH_ERR_NONPHYSICAL, "non-physical state (rho <= 0, stress not positive-definite or non-finite)");
    return CSH_OK;
}

void drop_graph(csh_grid* h)
{
    if (h->exec) (void)hipGraphExecDestroy(h->exec);
    h->exec = nullptr;
    h->g_nsteps = -1;
    h->g_mode = -1;
}

}  // namespace

int csh_fail(int code, const std::string& msg)
{
    csh_err_msg = msg;
    return code;
}

extern "C" int csh_init_state(csh_grid** out, int nx, int ny, double dx, double dy, int bc_x, int bc_y,
                              int dtype, const void* W, void* U, void* stream)
{
    if (!out) return csh_fail(CSH_ERR_ARG, "h is NULL");
    *out = nullptr;
    if (nx < 1 || ny < 1) return csh_fail(CSH_ERR_ARG, "nx and ny must be >= 1");
    if ((long long)nx * ny * (dtype == CSH_F32 ? 4 : 8) >= (1LL << 32))
        return csh_fail(CSH_ERR_ARG, "one plane of the state must be smaller than 4 GiB");
    if (!(dx > 0) || (ny > 1 && !(dy > 0))) return csh_fail(CSH_ERR_ARG, "dx, dy must be > 0");
    if ((bc_x != CSH_BC_PERIODIC && bc_x != CSH_BC_OUTFLOW) || (bc_y != CSH_BC_PERIODIC && bc_y != CSH_BC_OUTFLOW))
        return csh_fail(CSH_ERR_ARG, "bad boundary condition");
    if (dtype != CSH_F64 && dtype != CSH_F32) return csh_fail(CSH_ERR_ARG, "bad dtype");
    if (!W || !U) return csh_fail(CSH_ERR_ARG, "W and U must be device pointers");
    csh_grid* h = new csh_grid;
    h->nx = nx;
    h->ny = ny;
    h->dx = dx;
    h->dy = ny > 1 ? dy : 1.0;
    h->bcx = bc_x;
    h->bcy = bc_y;
    h->dtype = dtype;
    h->stream = static_cast<hipStream_t>(stream);
    split_rows(h);
    auto cleanup = [&](int code) {
        csh_destroy(h);
        return code;
    };
    if (hipMalloc(&h->slots, 3 * sizeof(Slot)) != hipSuccess || !(h->cell = csh::acquire_cell()))
        return cleanup(csh_fail(CSH_ERR_HIP, "allocation of the handle's scalars failed"));
    if (hipStreamCreateWithFlags(&h->capture, hipStreamNonBlocking) != hipSuccess)
        return cleanup(csh_fail(CSH_ERR_HIP, "hipStreamCreate failed"));
    const int64_t n = (int64_t)nx * ny;
    hipError_t e = csh::launch_reset(h->slots, 3, 0.0, h->stream);
    if (e == hipSuccess)
        e = dtype == CSH_F64 ? csh::launch_init<double>(static_cast<const double*>(W), static_cast<double*>(U), n, &h->cell->flag, h->stream)
                             : csh::launch_init<float>(static_cast<const float*>(W), static_cast<float*>(U), n, &h->cell->flag, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return cleanup(csh_fail(CSH_ERR_HIP, std::string("init: ") + hipGetErrorString(e)));
    *out = h;
    if (h->cell->flag) return csh_fail(CSH_ERR_NONPHYSICAL, "initial state not physical");
    return CSH_OK;
}

extern "C" int csh_set_state(csh_grid* h, const void* W, void* U)
{
    if (!h || !W || !U) return csh_fail(CSH_ERR_ARG, "NULL argument");
    const int64_t n = (int64_t)h->nx * h->ny;
    hipError_t e = csh::launch_clear_flag(&h->cell->flag, h->stream);
    if (e == hipSuccess)
        e = h->dtype == CSH_F64 ? csh::launch_init<double>(static_cast<const double*>(W), static_cast<double*>(U), n, &h->cell->flag, h->stream)
                                : csh::launch_init<float>(static_cast<const float*>(W), static_cast<float*>(U), n, &h->cell->flag, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("set_state: ") + hipGetErrorString(e));
    if (h->cell->flag) return csh_fail(CSH_ERR_NONPHYSICAL, "state not physical");
    return CSH_OK;
}

extern "C" int csh_set_scheme(csh_grid* h, int scheme)
{
    if (!h) return csh_fail(CSH_ERR_ARG, "h is NULL");
    if (scheme != CSH_SCHEME_MUSCL_HLL && scheme != CSH_SCHEME_KT && scheme != CSH_SCHEME_MUSCL_HLLC)
        return csh_fail(CSH_ERR_ARG, "unknown scheme");
    if (scheme == CSH_SCHEME_KT && h->ny == 1 && !h->kt_buf) {  // the 1-D stage buffer
        const size_t bytes = 6 * (size_t)h->nx * h->ny * (h->dtype == CSH_F64 ? 8 : 4);
        CSH_HIP(hipStreamSynchronize(h->stream));
        CSH_HIP(hipMalloc(&h->kt_buf, bytes));
    }
    if (scheme == CSH_SCHEME_KT && h->ny > 1) h->kt_plan = csh::kt_plan(h->nx, h->ny, h->dtype == CSH_F64);
    h->scheme = scheme;
    drop_graph(h);
    return CSH_OK;
}

extern "C" int csh_fourier_amplitudes(csh_grid* h, const void* U, double x0, double y0, double X, double Y,
                                      int m_max, double* A)
{
    if (!h || !U || !A) return csh_fail(CSH_ERR_ARG, "NULL argument");
    if (h->ny < 2) return csh_fail(CSH_ERR_ARG, "Fourier amplitudes need a 2-D grid");
    if (m_max < 1 || m_max > CSH_FOURIER_MAX_M) return csh_fail(CSH_ERR_ARG, "m_max must be in 1..CSH_FOURIER_MAX_M");
    if (!(X > 0) || !(Y > 0)) return csh_fail(CSH_ERR_ARG, "X and Y must be > 0");
    if (!h->fourier_ws) {
        CSH_HIP(hipMalloc(&h->fourier_ws, sizeof(double) * ((size_t)csh::kFourierBlocks * (1 + 2 * csh::kFourierMaxM) +
                                                            csh::kFourierMaxM)));
    }
    double* dA = h->fourier_ws + (size_t)csh::kFourierBlocks * (1 + 2 * csh::kFourierMaxM);
    auto run = [&](auto tag) {
        using T = decltype(tag);
        csh::FourierArgs<T> a{static_cast<const T*>(U), h->nx, h->ny, h->dx, h->dy, x0, y0, X, Y, m_max,
                              h->fourier_ws, dA};
        return csh::launch_fourier<T>(a, h->stream);
    };
    hipError_t e = h->dtype == CSH_F64 ? run(double{}) : run(float{});
    if (e == hipSuccess) e = hipMemcpyAsync(A, dA, sizeof(double) * m_max, hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("fourier: ") + hipGetErrorString(e));
    return CSH_OK;
}

extern "C" int csh_fourier_amplitudes_noalloc(csh_grid* h, const void* U, double x0, double y0, double X, double Y,
                                              int m_max, double* A_dev)
{
    if (!h || !U || !A_dev) return csh_fail(CSH_ERR_ARG, "NULL argument");
    if (h->ny < 2) return csh_fail(CSH_ERR_ARG, "Fourier amplitudes need a 2-D grid");
    if (m_max < 1 || m_max > CSH_FOURIER_MAX_M)
        return csh_fail(CSH_ERR_ARG, "m_max must be in 1..CSH_FOURIER_MAX_M (the static partial sums' limit)");
    if (!(X > 0) || !(Y > 0)) return csh_fail(CSH_ERR_ARG, "X and Y must be > 0");
    double* partials = nullptr;
    hipError_t e = csh::fourier_static_partials(&partials);
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("fourier (static partials): ") + hipGetErrorString(e));
    auto run = [&](auto tag) {
        using T = decltype(tag);
        csh::FourierArgs<T> a{static_cast<const T*>(U), h->nx, h->ny, h->dx, h->dy, x0, y0, X, Y, m_max,
                              partials, A_dev};
        return csh::launch_fourier<T>(a, h->stream);
    };
    e = h->dtype == CSH_F64 ? run(double{}) : run(float{});
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("fourier: ") + hipGetErrorString(e));
    return CSH_OK;
}

extern "C" int csh_set_potential(csh_grid* h, double vc, double rc, double x0, double y0)
{
    if (!h) return csh_fail(CSH_ERR_ARG, "h is NULL");
    if (vc != 0 && !(rc > 0)) return csh_fail(CSH_ERR_ARG, "rc must be > 0");
    h->vc = vc;
    h->rc = rc;
    h->x0 = x0;
    h->y0 = y0;
    drop_graph(h);
    return CSH_OK;
}

extern "C" int csh_step(csh_grid* h, double dt, const void* U, void* U_new)
{
    if (!h || !U || !U_new) return csh_fail(CSH_ERR_ARG, "NULL argument");
    if (U == U_new) return csh_fail(CSH_ERR_ARG, "U and U_new must be distinct buffers");
    if (!(dt >= 0)) return csh_fail(CSH_ERR_ARG, "dt must be >= 0");
    hipError_t e = h->dtype == CSH_F64 ? enqueue_step<double>(h, U, U_new, 0, dt, 0, 0, nullptr, h->stream)
                                       : enqueue_step<float>(h, U, U_new, 0, dt, 0, 0, nullptr, h->stream);
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("step: ") + hipGetErrorString(e));
    return CSH_OK;
}

extern "C" int csh_max_signal_speed(csh_grid* h, const void* U, double* s)
{
    if (!h || !U || !s) return csh_fail(CSH_ERR_ARG, "NULL argument");
    hipError_t e = enqueue_maxspeed(h, U, h->stream);
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("max_signal_speed: ") + hipGetErrorString(e));
    return read_rate(h, s);
}

extern "C" int csh_last_signal_speed(csh_grid* h, double* s)
{
    if (!h || !s) return csh_fail(CSH_ERR_ARG, "NULL argument");
    return read_rate(h, s);
}

extern "C" int csh_fluxes(csh_grid* h, double dt, const void* U, void* Fx, void* Fy)
{
    if (!h || !U || !Fx || (h->ny > 1 && !Fy)) return csh_fail(CSH_ERR_ARG, "NULL argument");
    if (h->scheme == CSH_SCHEME_KT) return csh_fail(CSH_ERR_ARG, "fluxes are those of the characteristic scheme");
    hipError_t e;
    if (h->dtype == CSH_F64) {
        auto a = base_args<double>(h);
        a.U = static_cast<const double*>(U);
        a.Fx = static_cast<double*>(Fx);
        a.Fy = static_cast<double*>(Fy);
        a.dt = dt;
        a.s_in = h->phase;
        e = csh::launch_step<double>(a, h->ny > 1, true, solver_of(h), h->stream);
    } else {
        auto a = base_args<float>(h);
        a.U = static_cast<const float*>(U);
        a.Fx = static_cast<float*>(Fx);
        a.Fy = static_cast<float*>(Fy);
        a.dt = dt;
        a.s_in = h->phase;
        e = csh::launch_step<float>(a, h->ny > 1, true, solver_of(h), h->stream);
    }
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("fluxes: ") + hipGetErrorString(e));
    return CSH_OK;
}

namespace {

hipError_t enqueue_run(csh_grid* h, int nsteps, double cfl, double t_end, void* U, void* Uw, double* dt_log,
                       const double* dts, hipStream_t s)
{
    h->phase = 0;
    hipError_t e = enqueue_maxspeed(h, U, s);  // rate of the initial state into slot 0, t = 0
    for (int k = 0; k < nsteps && e == hipSuccess; ++k) {
        void* in = (k % 2 == 0) ? U : Uw;
        void* outp = (k % 2 == 0) ? Uw : U;
        double* lg = dt_log ? dt_log + k : nullptr;
        const double* di = dts ? dts + k : nullptr;
        const int dev = dts ? 0 : 1;
        e = h->dtype == CSH_F64 ? enqueue_step<double>(h, in, outp, dev, 0, cfl, t_end, lg, s, di)
                                : enqueue_step<float>(h, in, outp, dev, 0, cfl, t_end, lg, s, di);
    }
    if (e == hipSuccess && nsteps % 2 == 1) {
        const int64_t n = 6LL * h->nx * h->ny;
        e = h->dtype == CSH_F64 ? csh::launch_copy<double>(static_cast<double*>(Uw), static_cast<double*>(U), n, s)
                                : csh::launch_copy<float>(static_cast<float*>(Uw), static_cast<float*>(U), n, s);
    }
    return e;
}

// nsteps CFL steps keeping every state: step k reads the previous step's
// output (U0 for the first) and writes slot k of states
hipError_t enqueue_run_states(csh_grid* h, int nsteps, double cfl, const void* U0, void* states, double* dt_log,
                              hipStream_t s)
{
    h->phase = 0;
    hipError_t e = enqueue_maxspeed(h, U0, s);  // rate of the initial state into slot 0, t = 0
    const size_t bytes = 6 * (size_t)h->nx * h->ny * (h->dtype == CSH_F64 ? sizeof(double) : sizeof(float));
    char* base = static_cast<char*>(states);
    for (int k = 0; k < nsteps && e == hipSuccess; ++k) {
        const void* in = k == 0 ? U0 : base + (size_t)(k - 1) * bytes;
        void* outp = base + (size_t)k * bytes;
        double* lg = dt_log ? dt_log + k : nullptr;
        e = h->dtype == CSH_F64 ? enqueue_step<double>(h, in, outp, 1, 0, cfl, 0.0, lg, s)
                                : enqueue_step<float>(h, in, outp, 1, 0, cfl, 0.0, lg, s);
    }
    return e;
}

// Short 1-D grids take their whole run in one launch, which a recorded graph of a
// launch per step does not match (us per step: 256 cells 1.7 against 3.3, 960 cells 3.2
// against 3.4, with the Kurganov-Tadmor step 4.0 against 5.9, with HLLC 3.5 either way).
bool one_launch(const csh_grid* h)
{
    return h->ny == 1 && h->nx <= csh::kLineCells;
}

template <typename T>
hipError_t enqueue_line_run(csh_grid* h, int nsteps, double cfl, double t_end, const void* U0, void* U,
                            void* states, double* dt_log, const double* dts)
{
    csh::LineArgs<T> a{};
    a.U0 = static_cast<const T*>(U0);
    a.U = static_cast<T*>(U);
    a.states = static_cast<T*>(states);
    a.nx = h->nx;
    a.bcx = h->bcx;
    a.nsteps = nsteps;
    a.dx = h->dx;
    a.dy = h->dy;
    a.cfl = cfl;
    a.t_end = t_end;
    a.dts = dts;
    a.dt_log = dt_log;
    a.slots = h->slots;
    h->phase = a.s_out = nsteps % 3;
    a.flag = &h->cell->flag;
    a.vc2 = h->vc * h->vc;
    a.rc2 = h->rc * h->rc;
    a.x0 = h->x0;
    a.y0 = h->y0;
    return csh::launch_line_run<T>(a, h->scheme == CSH_SCHEME_KT ? 2 : solver_of(h), h->stream);
}

int line_run(csh_grid* h, int nsteps, double cfl, double t_end, const void* U0, void* U, void* states,
             double* dt_log, const double* dts)
{
    const hipError_t e = h->dtype == CSH_F64
                             ? enqueue_line_run<double>(h, nsteps, cfl, t_end, U0, U, states, dt_log, dts)
                             : enqueue_line_run<float>(h, nsteps, cfl, t_end, U0, U, states, dt_log, dts);
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("run: ") + hipGetErrorString(e));
    return CSH_OK;
}

// Whether a run's steps are replayed as a recorded graph.  The host enqueues a
// launch in ~3 us and the device takes ~0.4 us longer between two of them than
// between two nodes of a graph, but recording 100 steps takes 0.4-0.5 ms: from
// 4 strip rows per SIMD (a step of 13 us, 512^2) the plain launches are as fast
// (100 steps of 512^2: 1389 against 1396 us, 64^2: 549 against 509 us) and the
// first run is spared the recording (1480 against 1750 us).
// Nor is a run of up to four launches worth it: a graph's launch takes as long as those
// of about six kernels, and its log is copied by one more (us per run, recorded / launched
// one by one, alone: one step of 64^2 45 / 25, of a 1-D grid of 961 cells 45 / 25, four
// steps 47 / 40 and 44 / 33, eight 64 / 71 and 52 / 65).
bool worth_recording(const csh_grid* h, int nsteps)
{
    const int launches = h->scheme == CSH_SCHEME_KT && h->ny == 1 ? 2 : 1;  // of a step
    return nsteps > 4 / launches && (long)((h->nx + csh::kStrip - 1) / csh::kStrip) * h->ny <= 4L * 1024;
}

// All steps of csh_run_cfl (mode 0, lg: the log or null) or csh_run_dts (mode 1,
// lg: the timesteps): launched one by one, or replayed from a graph recorded once
// per argument set.  The graph logs into the handle's own buffer, so that it
// serves every log the caller passes.
int run_steps(csh_grid* h, int mode, int nsteps, double cfl, double t_end, void* U, void* U_work, const void* lg)
{
    auto enqueue = [&](const void* l, hipStream_t s) {
        return mode == 0 ? enqueue_run(h, nsteps, cfl, t_end, U, U_work, (double*)l, nullptr, s)
                         : enqueue_run(h, nsteps, 1.0, 0.0, U, U_work, nullptr, (const double*)l, s);
    };
    if (!worth_recording(h, nsteps)) {
        const hipError_t e = enqueue(lg, h->stream);
        if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("run: ") + hipGetErrorString(e));
        return CSH_OK;
    }
    const bool log = mode == 0 && lg;
    if (log && h->log_n < nsteps) {
        CSH_HIP(hipStreamSynchronize(h->stream));
        drop_graph(h);
        if (h->log) (void)hipFree(h->log);
        h->log = nullptr;
        h->log_n = 0;
        CSH_HIP(hipMalloc(&h->log, sizeof(double) * (size_t)nsteps));
        h->log_n = nsteps;
    }
    const void* l = log ? h->log : lg;
    const bool same = h->exec && h->g_mode == mode && h->g_nsteps == nsteps && h->g_cfl == cfl &&
                      h->g_tend == t_end && h->g_U == U && h->g_W == U_work && h->g_log == l;
    if (!same) {
        drop_graph(h);
        hipGraph_t g = nullptr;
        CSH_HIP(hipStreamBeginCapture(h->capture, hipStreamCaptureModeThreadLocal));
        hipError_t e = enqueue(l, h->capture);
        hipError_t e2 = hipStreamEndCapture(h->capture, &g);
        if (e != hipSuccess || e2 != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            return csh_fail(CSH_ERR_HIP, std::string("run capture: ") + hipGetErrorString(e != hipSuccess ? e : e2));
        }
        e = hipGraphInstantiate(&h->exec, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e != hipSuccess) {
            h->exec = nullptr;
            return csh_fail(CSH_ERR_HIP, std::string("run instantiate: ") + hipGetErrorString(e));
        }
        h->g_mode = mode;
        h->g_nsteps = nsteps;
        h->g_cfl = cfl;
        h->g_tend = t_end;
        h->g_U = U;
        h->g_W = U_work;
        h->g_log = l;
    }
    CSH_HIP(hipGraphLaunch(h->exec, h->stream));
    h->phase = nsteps % 3;
    if (log) CSH_HIP(csh::launch_copy<double>(h->log, (double*)lg, nsteps, h->stream));
    return CSH_OK;
}

}  // namespace

extern "C" int csh_run_cfl(csh_grid* h, int nsteps, double cfl, double t_end, void* U, void* U_work,
                           double* dt_log)
{
    if (!h || !U || !U_work) return csh_fail(CSH_ERR_ARG, "NULL argument");
    if (U == U_work) return csh_fail(CSH_ERR_ARG, "U and U_work must be distinct");
    if (nsteps < 0 || !(cfl > 0)) return csh_fail(CSH_ERR_ARG, "nsteps >= 0 and cfl > 0 required");
    if (nsteps == 0) return CSH_OK;
    if (one_launch(h)) return line_run(h, nsteps, cfl, t_end, U, U, nullptr, dt_log, nullptr);
    return run_steps(h, 0, nsteps, cfl, t_end, U, U_work, dt_log);
}

extern "C" int csh_run_cfl_states(csh_grid* h, int nsteps, double cfl, const void* U0, void* states,
                                  double* dt_log)
{
    if (!h || !U0 || !states) return csh_fail(CSH_ERR_ARG, "NULL argument");
    if (U0 == states) return csh_fail(CSH_ERR_ARG, "U0 must not be the state array");
    if (nsteps < 0 || !(cfl > 0)) return csh_fail(CSH_ERR_ARG, "nsteps >= 0 and cfl > 0 required");
    if (nsteps == 0) return CSH_OK;
    if (one_launch(h)) return line_run(h, nsteps, cfl, 0.0, U0, nullptr, states, dt_log, nullptr);
    // enqueued directly: the state array is usually new at every call, and at
    // the sizes these runs serve a graph replay is no faster than the launches
    const hipError_t e = enqueue_run_states(h, nsteps, cfl, U0, states, dt_log, h->stream);
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("run_cfl_states: ") + hipGetErrorString(e));
    return CSH_OK;
}

extern "C" int csh_run_dts(csh_grid* h, int nsteps, const double* dts, void* U, void* U_work)
{
    if (!h || !U || !U_work || (nsteps > 0 && !dts)) return csh_fail(CSH_ERR_ARG, "NULL argument");
    if (U == U_work) return csh_fail(CSH_ERR_ARG, "U and U_work must be distinct");
    if (nsteps < 0) return csh_fail(CSH_ERR_ARG, "nsteps >= 0 required");
    if (nsteps == 0) return CSH_OK;
    if (one_launch(h)) return line_run(h, nsteps, 1.0, 0.0, U, U, nullptr, nullptr, dts);
    return run_steps(h, 1, nsteps, 0.0, 0.0, U, U_work, dts);
}

extern "C" int csh_destroy(csh_grid* h)
{
    if (!h) return CSH_OK;
    if (h->stream || h->slots) (void)hipStreamSynchronize(h->stream);
    drop_graph(h);
    if (h->capture) (void)hipStreamDestroy(h->capture);
    if (h->slots) (void)hipFree(h->slots);
    csh::release_cell(h->cell);
    if (h->adj_ws) (void)hipFree(h->adj_ws);
    if (h->log) (void)hipFree(h->log);
    if (h->kt_buf) (void)hipFree(h->kt_buf);
    if (h->fourier_ws) (void)hipFree(h->fourier_ws);
    delete h;
    return CSH_OK;
}

// adjoint entry points: implemented with the adjoint kernels
size_t csh_adjoint_workspace_doubles(int nx, int ny);
int csh_adjoint_impl(csh_grid_view v, double dt, const void* U, const void* lam_next, void* lam, double* ws,
                     hipStream_t s);
int csh_init_adjoint_impl(int64_t n, const void* W, const void* lamU, void* lamW, hipStream_t s);

extern "C" int csh_adjoint_step(csh_grid* h, double dt, const void* U, const void* lam_next, void* lam)
{
    if (!h || !U || !lam_next || !lam) return csh_fail(CSH_ERR_ARG, "NULL argument");
    if (h->dtype != CSH_F64) return csh_fail(CSH_ERR_ARG, "the adjoint is FP64 only");
    if (h->scheme != CSH_SCHEME_MUSCL_HLL)
        return csh_fail(CSH_ERR_ARG, "the adjoint is that of the characteristic scheme with the HLL flux");
    if (lam == lam_next || lam == U) return csh_fail(CSH_ERR_ARG, "lam must not alias U or lam_next");
    if (!(dt >= 0)) return csh_fail(CSH_ERR_ARG, "dt must be >= 0");
    const size_t need = csh_adjoint_workspace_doubles(h->nx, h->ny);
    if (h->adj_ws_n < need) {
        CSH_HIP(hipStreamSynchronize(h->stream));
        if (h->adj_ws) (void)hipFree(h->adj_ws);
        h->adj_ws = nullptr;
        h->adj_ws_n = 0;
        CSH_HIP(hipMalloc(&h->adj_ws, need * sizeof(double)));
        h->adj_ws_n = need;
    }
    csh_grid_view v{h->nx, h->ny, h->bcx, h->bcy, h->dx, h->dy, h->vc, h->rc, h->x0, h->y0};
    return csh_adjoint_impl(v, dt, U, lam_next, lam, h->adj_ws, h->stream);
}

extern "C" int csh_init_state_adjoint(csh_grid* h, const void* W, const void* lam_U, void* lam_W)
{
    if (!h || !W || !lam_U || !lam_W) return csh_fail(CSH_ERR_ARG, "NULL argument");
    if (h->dtype != CSH_F64) return csh_fail(CSH_ERR_ARG, "the adjoint is FP64 only");
    return csh_init_adjoint_impl((int64_t)h->nx * h->ny, W, lam_U, lam_W, h->stream);
}
