// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace csh {

// Device scalars of the timestep reduction.  Step n reads slot n % 3 (the
// rate s of its input and the time t), accumulates the rate of its output
// into slot (n + 1) % 3 and clears slot (n + 2) % 3 for the step after.
// The rate is kept in kRateParts partial maxima, each on a 128-byte line of its
// own, workgroup b adding to part b % kRateParts: workgroups are dealt
// round-robin to the 8 XCDs, so the atomics on a part come from one XCD and
// stay in its L2.  With one word for the whole launch every wavefront's atomic
// moved that word between the L2s, ~10 ns each at the end of the launch
// (512^2: 576 wavefronts, the last ended at 15.4 us of a 23.5 us step).
constexpr int kRateParts = 8;

struct Slot {
    double t;   // simulation time of the state this slot describes
    double dt;  // timestep a multi-stage step chose in its first stage
    double pad[14];
    struct {
        unsigned long long bits;  // max CFL rate as the bit pattern of a positive double
        unsigned long long pad[15];
    } part[kRateParts];
};

// What a handle's kernels tell the host, in pinned memory the kernels write
// directly: the host reads it after a stream synchronisation, with no copy (two
// small copies to pageable memory had cost ~25 us of a 47 us host-stepped step
// at 251 x 187).  The flag is written only when a non-physical state is met.
struct alignas(64) HostCell {
    double rate;  // written by launch_publish
    int flag;     // 1 once a non-physical state was seen
};

// A cell for one handle (null if out of memory), flag 0, and its return once
// the handle's stream is idle.  Thread-safe; pages of 64 cells, each freed with
// its last cell, but for one page kept for the next handle (a pinned allocation
// takes ~0.3 ms, more than the rest of making a handle).
HostCell* acquire_cell();
void release_cell(HostCell* cell);

// Sets the flag (any lane, any number of times).
__device__ __forceinline__ void raise_flag(int* flag)
{
    __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Clears a slot's rate: threads 0 .. kRateParts - 1 of one workgroup.
__device__ __forceinline__ void slot_clear(Slot& sl, int thread)
{
    if (thread < kRateParts) sl.part[thread].bits = 0ull;
}

// Adds one workgroup's (or wavefront's) rate to a slot: one lane calls this.
// Positive doubles order like their bit patterns.
__device__ __forceinline__ void slot_add(Slot& sl, unsigned workgroup, double s)
{
    atomicMax(&sl.part[workgroup % kRateParts].bits, (unsigned long long)__double_as_longlong(s));
}

constexpr int kStrip = 60;  // output columns per wavefront (64 lanes, 2 halo lanes per side)
constexpr int kWaves = 4;   // wavefronts per workgroup of the sweep kernels

template <typename T>
struct StepArgs {
    const T* U;   // input state [6][ny][nx]
    T* Unew;      // output state (step) -- may not alias U
    T* Fx;        // face fluxes (flux mode): [6][ny][nx+1], column i = face i-1/2
    T* Fy;        // [6][ny+1][nx], row j = face j-1/2
    int nx, ny, bcx, bcy;
    double dx, dy;
    int nstrips, nsegs, ty;  // strips of kStrip columns, segments of ty rows
    int tw;                  // 2-D sweep: rows per wavefront of a segment's ty + 2
    double dt;               // timestep when dev_dt == 0
    int dev_dt;              // 1: dt = min(cfl / s, t_end - t) from slots[s_in]
    double cfl, t_end;       // t_end <= 0: no end time
    Slot* slots;
    int s_in, s_out, s_reset;
    double* dt_log;          // if set, receives the timestep used
    const double* dt_in;     // if set (and dev_dt == 0), the timestep is read from here
    double vc2, rc2, x0, y0; // external flat-rotation-curve potential (vc2 == 0: none)
    int* flag;               // raised if an output cell is not physical
    const T* Ubase;          // two-stage schemes: state the stage update starts from (null: U)
};

// solver: 0 HLL, 1 HLLC
template <typename T>
hipError_t launch_step(const StepArgs<T>& a, bool twod, bool fluxes, int solver, hipStream_t s);

template <typename T>
hipError_t launch_init(const T* W, T* U, int64_t n, int* flag, hipStream_t s);

template <typename T>
hipError_t launch_maxspeed(const T* U, int nx, int ny, double dx, double dy, Slot* slot, int* flag,
                           hipStream_t s);

hipError_t launch_reset(Slot* slots, int nslots, double t0, hipStream_t s);

// In stream order: the slot's rate to the host's cell; the flag cleared.
hipError_t launch_publish(const Slot* slot, HostCell* cell, hipStream_t s);
hipError_t launch_clear_flag(int* flag, hipStream_t s);

// Kurganov-Tadmor stage on a 1-D grid: first (half step into the stage
// buffer, records dt in slots[s_in].dt) or final (full step from Ubase with
// the stage state's fluxes)
template <typename T>
hipError_t launch_kt(const StepArgs<T>& a, bool final_stage, hipStream_t s);

// Kurganov-Tadmor step on a 2-D grid, both stages in one launch: its kernel (a
// workgroup or a wavefront per segment) and its rows per segment, chosen once for a
// grid; the arguments' own decomposition fields are ignored
struct KtPlan {
    bool block;
    int rows;
};
KtPlan kt_plan(int nx, int ny, bool f64);
template <typename T>
hipError_t launch_kt_fused(StepArgs<T> a, KtPlan plan, hipStream_t s);

// Whole runs of a 1-D grid of at most kLineCells cells in one launch.  U: in
// place (null: the input U0 is left); states: if set, step k's result goes to
// states + 6 nx k; dts: if set, the given timesteps, else cfl / s, clipped at
// t_end (<= 0: none).  The slots are left as after nsteps single steps.
constexpr int kLineCells = 16 * kStrip;

template <typename T>
struct LineArgs {
    const T* U0;
    T *U, *states;
    int nx, bcx, nsteps;
    double dx, dy, cfl, t_end;
    const double* dts;
    double* dt_log;
    Slot* slots;
    int s_out;
    int* flag;
    double vc2, rc2, x0, y0;
};

// scheme: 0 characteristic with HLL, 1 with HLLC, 2 Kurganov-Tadmor
template <typename T>
hipError_t launch_line_run(const LineArgs<T>& a, int scheme, hipStream_t s);

template <typename T>
hipError_t launch_copy(const T* src, T* dst, int64_t n, hipStream_t s);

}  // namespace csh
