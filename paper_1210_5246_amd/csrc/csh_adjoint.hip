// Adjoint of one sweep at frozen timestep (FP64): lam^n = (d S_dt / d U^n)^T lam^{n+1}.
//
// 2-D grids: one kernel, adjoint_fused_kernel: blocks of cells whose face states,
// flux adjoints, face-state reverse pass and sums stay in registers and LDS.
//
// 1-D grids: the forward step reads primitive states at "extended" cells
// e = i, i in [-1, nx], whose values come from the mapped cells map(e) of the
// boundary conditions; each extended cell builds its face states from itself
// and its two neighbours; every face flux uses the high state of one extended
// cell and the low state of the next.  The reverse pass follows the same
// structure in four kernels, with fixed slots instead of atomics so the result
// is deterministic:
//   1. faces:  recompute the face states of every extended cell -> FS
//   2. hll:    per face, lam' = K^T lam^{n+1} (kick), flux adjoint
//              dt/dx (lam'_{i+1} - lam'_i), HLL vjp -> adjoints of the two face
//              states, each written to its one slot in FSb
//   3. cells:  per extended cell, the vjp of its face-state computation; a
//              wavefront covers 64 consecutive cells and sums self + the right
//              neighbour's left share + the left neighbour's right share by
//              lane shifts into one value per padded position (XS)
//   4. gather: per interior cell, sum the XS of the padded positions that the
//              boundary mapping sends to this cell, chain through W(U) and add
//              lam' itself.
// (tests/host holds that scheme with a y part, the CPU reference of the 2-D kernel.)
//
// The kernels take their workgroup numbers XCD-aware (xcd_block), so blocks that
// share halo cells sit in the same L2.
#include <string>

#include "csh_adjoint.h"
#include "csh_api_util.h"

namespace csh {

// ---- kernels ----------------------------------------------------------------------------------------

// Stages 1, 2 and 4 of 1-D grids, a thread per cell.
template <int STAGE>
__global__ __launch_bounds__(256) void adjoint_kernel(AdjArgs a)
{
    // cell counts stay below 2^31 (a plane is smaller than 4 GiB): 32-bit index arithmetic
    const unsigned t = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (STAGE == 4) {  // interior cells
        if (t < (unsigned)a.nx) gather_cell(a, (int)t);
        return;
    }
    if (t >= (unsigned)a.nx + 2) return;  // extended cells
    if (STAGE == 1) faces_cell(a, (int)t - 1);
    if (STAGE == 2) hll_cell(a, (int)t - 1);
}

// Stage 3, summed per padded position: a wavefront covers the extended cells
// base .. base + 63 (base = 62 w - 3) and
// writes the padded positions of its lanes 1..62; lanes outside the extended
// range contribute zero.  The summation order is that of a per-position sum of
// slots: self, then the left share of the cell to the right, then the right
// share of the cell to the left.
constexpr int kXsOwned = 62;

__global__ __launch_bounds__(256) void adjoint_xsum_kernel(AdjArgs a)
{
    const int lane = threadIdx.x & 63;
    const long w = (long)xcd_block(blockIdx.x, gridDim.x) * 4 + wave_in_block();
    if (w >= (a.nx + 4 + kXsOwned - 1) / kXsOwned) return;  // uniform per wavefront
    const int i = (int)w * kXsOwned - 3 + lane;
    P b0 = zero_p(), bl = zero_p(), br = zero_p();
    if (i >= -1 && i <= a.nx) cells_x_vjp(a, i, b0, bl, br);
    const P l = lane_shift<+1>(bl), r = lane_shift<-1>(br);  // from the cells at i + 1, i - 1
    const P sum = {b0.r + l.r + r.r,       b0.u + l.u + r.u,       b0.v + l.v + r.v,
                   b0.pxx + l.pxx + r.pxx, b0.pxy + l.pxy + r.pxy, b0.pyy + l.pyy + r.pyy};
    if (lane >= 1 && lane <= kXsOwned && i >= -2 && i <= a.nx + 1)
        store_p(a.XS, (size_t)(a.nx + 4), 0, (size_t)(i + 2), sum);
}

// The reverse pass of 2-D grids, one launch.  A workgroup holds a block of
// BX x 16 cells (a thread each; a cell outside the grid is a virtual one: the
// wrapped cell on a periodic axis, else the ghost cell, with lam' = 0) and outputs
// its inner (BX - 4) x 12.  Per cell: the face states (states of the block and a
// ring in LDS); the flux adjoints of its high x and y faces through HLL into the
// adjoints of the face states on both sides; the face-state reverse pass; the sum
// of what lands on each position, on outflow axes folded onto the boundary cells;
// W(U) reverse and lam'.  x neighbours exchange by lane shifts (a shift that
// crosses from one row of the block to the next lands on a cell whose value is not
// used or is zero), y neighbours through LDS, where a slot read by one thread only
// is overwritten by it: four barriers (a fifth in the blocks that fold a y boundary).
//
// Two launches with the face-state adjoints in between (192 B per cell written and
// read with a ring) moved 663 B per cell-step, 49 us at 512^2 whatever their
// instruction count; here the state, lam^{n+1} and lam^n are all that is moved
// (131 x 93 16.9 -> 7.9 us, 300 x 200 21.1 -> 11.7, 512^2 51.2 -> 38.6).  Bound by
// FP64 issue (VALU busy 0.49: ~1800 instructions a thread, 256 threads for 144
// outputs) and by the latency of its phases at two wavefronts per SIMD (230
// registers: values are put into LDS as soon as they are known and read again after
// the fluxes; kept through the reverse pass they spilled 44 B a thread, 131 x 93
// 8.5 us, 400^2 23.2 against 21.3).
template <int BX>
__global__ __launch_bounds__(BX * kF_Y, 2) void adjoint_fused_kernel(AdjArgs a, int tiles_x)
{
    using Thread = AdjointThread<BX>;
    __shared__ double S[Thread::kStates], Y[Thread::kRows], M[Thread::kRows];
    Thread t(a, S, Y, M, xcd_block(blockIdx.x, gridDim.x), tiles_x, (int)threadIdx.x);
    t.load();
    __syncthreads();
    t.faces();
    const P low = t.x_face(lane_shift<+1>(t.f.xlo), lane_shift<+1>(t.lam));
    t.fb.xlo = lane_shift<-1>(low);
    __syncthreads();
    t.y_face();
    __syncthreads();
    t.shares();
    t.land_x(lane_shift<+1>(t.left), lane_shift<-1>(t.right));
    __syncthreads();
    t.land_y();
    if (t.folds_x()) {
        const P l1 = lane_shift<-1>(t.self), r1 = lane_shift<+1>(t.self);
        t.fold_x(l1, lane_shift<-1>(l1), r1, lane_shift<+1>(r1));
    }
    if (t.folds_y()) {
        t.put_total();
        __syncthreads();
        t.fold_y();
    }
    t.store();
}

__global__ __launch_bounds__(256) void init_adjoint_kernel(const double* W, const double* lamU, double* lamW, int64_t n)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    const P w = {W[c], W[n + c], W[2 * n + c], W[3 * n + c], W[4 * n + c], W[5 * n + c]};
    P wb = zero_p();
    to_cons_vjp(w, load_cons<double>(lamU, (size_t)n, (size_t)c), wb);
    lamW[c] = wb.r;
    lamW[n + c] = wb.u;
    lamW[2 * n + c] = wb.v;
    lamW[3 * n + c] = wb.pxx;
    lamW[4 * n + c] = wb.pxy;
    lamW[5 * n + c] = wb.pyy;
}

}  // namespace csh

size_t csh_adjoint_workspace_doubles(int nx, int ny)
{
    return ny > 1 ? 0 : csh::workspace_1d(nx);
}

int csh_adjoint_impl(csh_grid_view v, double dt, const void* U, const void* lam_next, void* lam, double* ws,
                     hipStream_t s)
{
    using namespace csh;
    const bool twod = v.ny > 1;
    AdjArgs a{};
    a.nx = v.nx;
    a.ny = v.ny;
    a.bcx = v.bcx;
    a.bcy = v.bcy;
    a.dx = v.dx;
    a.dy = v.dy;
    a.dt = dt;
    set_step_factors(a);
    a.vc2 = v.vc * v.vc;
    a.rc2 = v.rc * v.rc;
    a.x0 = v.x0;
    a.y0 = v.y0;
    a.U = static_cast<const double*>(U);
    a.lam1 = static_cast<const double*>(lam_next);
    a.lam0 = static_cast<double*>(lam);
    if (twod) {
        // Blocks of 16 columns, two on a CU at a time, or of 32, one on a CU: the wider
        // ones trace fewer cells twice (28 x 12 outputs of 32 x 16 cells against
        // 12 x 12 of 16 x 16), the narrower ones overlap two blocks' barriers.  A round
        // of them takes 8 to 10 and 10.6 us; the launch takes the fewer (us, 16 / 32 columns:
        // 131 x 93 7.9 / 10.8, 300 x 200 11.8 / 11.6, 400^2 24.3 / 21.4, 480^2
        // 32.5 / 31.4, 512^2 38.8 / 41.7, 560^2 41.0 / 41.6, 1024^2 122 / 130).
        auto tiles = [&](int n, int o) { return (long)((n + o - 1) / o); };
        const long n16 = tiles(v.nx, 12) * tiles(v.ny, kF_OY), n32 = tiles(v.nx, 28) * tiles(v.ny, kF_OY);
        if (10 * ((n16 + 511) / 512) <= 13 * ((n32 + 255) / 256))
            adjoint_fused_kernel<16><<<(unsigned)n16, 16 * kF_Y, 0, s>>>(a, (int)tiles(v.nx, 12));
        else
            adjoint_fused_kernel<32><<<(unsigned)n32, 32 * kF_Y, 0, s>>>(a, (int)tiles(v.nx, 28));
    } else {
        set_workspace_1d(a, ws);
        const unsigned be = (unsigned)(((size_t)v.nx + 2 + 255) / 256), bi = (unsigned)(((size_t)v.nx + 255) / 256);
        const unsigned bx = (unsigned)(((a.nx + 4 + kXsOwned - 1) / kXsOwned + 3) / 4);
        adjoint_kernel<1><<<be, 256, 0, s>>>(a);
        adjoint_kernel<2><<<be, 256, 0, s>>>(a);
        adjoint_xsum_kernel<<<bx, 256, 0, s>>>(a);
        adjoint_kernel<4><<<bi, 256, 0, s>>>(a);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("adjoint_step: ") + hipGetErrorString(e));
    return CSH_OK;
}

int csh_init_adjoint_impl(int64_t n, const void* W, const void* lamU, void* lamW, hipStream_t s)
{
    csh::init_adjoint_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(
        static_cast<const double*>(W), static_cast<const double*>(lamU), static_cast<double*>(lamW), n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return csh_fail(CSH_ERR_HIP, std::string("init_state_adjoint: ") + hipGetErrorString(e));
    return CSH_OK;
}
