// Internal structures shared by the kernels and the host engine of libpoisson.
// Nothing here is part of the C ABI (include/poisson.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pois {

constexpr int kHistCap = 256;      // residual-history entries kept per solve
constexpr int kPartialStride = 8;  // doubles per set of partial sums (one set per block or per unit of work)
constexpr int kMaxSetupBlocks = 4096;
constexpr unsigned kArriveGroups = 32;  // counters a launch's blocks arrive at (last_block) ...
constexpr int kArriveStep = 4;          // ... in every fourth set of partial sums
constexpr int kStageTail = 3;  // see SolveState::stage
constexpr int kMaxInnerPerStep = 1 << 20;  // FP32 inner sweeps per refinement step: bounded by max_iter

// Grid description passed by value to every kernel.  Uniform over a batch:
// all solves of one launch share the grid.
struct GridArgs {
    int nx, ny, nz;
    int nxh;           // nx / 2 (complex columns of a row pair view)
    long long n;       // cells
    double ihx2, ihy2, ihz2;  // 1 / h_d^2
    int coef;          // face-coefficient mode
    int weight;        // residual multiplier mode
    int bcx;           // 0 periodic in x; 1 zero-flux walls at both ends of x
};

// Per-solve state, resident in device memory.  Zeroed by the init kernel and
// written by one block of a launch at a time (the last to arrive, when the others
// have read what they need); every sweep kernel reads `done` first and returns at
// once when the solve is over, so that unrolled iteration sequences stop doing
// work after convergence.
struct SolveState {
    // parameters (init kernel)
    double tol;
    double inner_tol;
    double inner_goal;  // inner stop of the current refinement step (decide_outer)
    int max_iter;
    int max_outer;
    int precision;
    unsigned arrive;    // groups of the running launch's blocks that have all arrived
                        // (last_block); 0 between launches
    // setup results
    double b_mean;
    double b_sumsq;     // sum b^2 (for the FP32 scale only)
    double rho_min, rho_max;
    int bad;            // non-finite or non-positive input seen
    // outer (FP64) iteration
    int iter;           // FP64 path: current iteration; FP32 path: current outer step
    int done;           // solve finished (any status)
    int status;         // POISSON_* code
    double b_norm;      // ||b - mean b||
    double r_norm;      // last FP64 residual norm
    double rel;         // last relative residual
    double rel0;        // relative residual of the first FP64 evaluation
    double p_shift;     // mean of the incoming p, removed by the first update
    double p_sum;       // sum p and sum p^2 of the last iterate whose residual was taken
    double p_sumsq;
    int p_fixed;        // p_shift already removed
    // FP32 inner iteration.  stage: 0 the next FP64 outer residual is due, 1 inner
    // FP32 sweeps run, 2 the FP64 update is due, 3 (kStageTail) the rest of the
    // first inner sweep is due after an outer residual that also produced that
    // sweep's transformed weighted residual; each kernel acts only on the solves
    // in its stage, so solves at different stages share one launch sequence
    int stage;
    int inner_iter;     // inner iteration within the current outer step
    int inner_done;
    int inner_total;
    int inner_last;     // inner-sweep launches the last finished outer step used
    int p1_work;        // launches of the residual sweep P1 that did their work
    int since_best;
    int stop_next;      // the inner phase ends after the update of the iteration in progress:
                        // the next inner residual sweep evaluates nothing and closes the phase
    int upd_due;        // the last inner evaluation went on with the phase and its update (the
                        // y, z, y and x sweeps) has not run yet: the next inner residual sweep
                        // idles until it has (the x sweep clears it)
    int checked;        // the last outer residual was a check (sums alone) that did not end the
                        // solve: `rel` is the residual of the current p, no update is pending
    double inv_s;       // r32 = r * inv_s (a power of two)
    double rhs_mean32;  // mean of r32, removed inside the inner sweeps
    double rhs_norm32;  // ||r32 - mean||
    double rel_in;
    double best_in;
    double hist[kHistCap];
};

// What a finished solve leaves to k_fixup: p = 0 where b - mean(b) is 0, and the
// mean of the incoming p, which the first update removes, where none ran (iter ==
// 0 on both paths).
__host__ __device__ inline bool solution_is_zero(const SolveState& st) {
    return st.b_norm == 0.0 && st.done && st.status == POISSON_OK;
}
__host__ __device__ inline bool fixup_due(const SolveState& st) {
    return st.status != POISSON_EDOMAIN && (solution_is_zero(st) || (st.iter == 0 && st.p_shift != 0.0));
}

// Per-solve device pointers (a batch launch indexes these by blockIdx.y).
struct Slot {
    double tol;       // relative-residual target of this solve
    const double* rho;
    const double* b;
    double* p;
    double* W;        // FP64 spectral workspace, n values
    float* rho32;     // FP32 copies / workspace (FP32_REFINE only)
    float* r32;
    float* d32;
    float* W32;
    double* partial;  // partial sums: kPartialStride doubles per block or per tile / line group
    SolveState* st;
};

// Device tables for one grid, shared by every solve of that grid.
struct Tables {
    const double2* twx; const double2* twy; const double2* twz;  // exp(-2 pi i t/N), FP64
    const float2* twx32; const float2* twy32; const float2* twz32;
    // symbols: -4 sin^2(pi k/N)/h^2; along x between walls -4 sin^2(pi k/(2N))/h^2
    const double* lamx; const double* lamy; const double* lamz;
    const float* lamx32; const float* lamy32; const float* lamz32;
    // walls in x: exp(-i pi k/(2 Nx)), the twiddles of the cosine transform
    const double2* twcx; const float2* twcx32;
};

// Launch geometry of the sweeps of one grid (host side).
struct Geometry {
    int blocks_x;      // row-pair line groups of the x sweep (most blocks P1 can use)
    int blocks_pt;     // pointwise kernels
    int blocks_outer;  // FP64 outer residual
    int max_blocks;    // capacity of the partial-sum array, in sets
    float share;       // fraction of the chip's resident blocks the persistent sweeps take
};

// ---- launchers (poisson_kernels.hip) ----------------------------------------
// Every launcher enqueues on `stream` for `nslots` solves described by the
// device array `slots`.  They return hipSuccess or the launch error.
Geometry make_geometry(const GridArgs& g);
bool length_supported(int n);

// Initialises the state of each slot (tolerance from Slot::tol).
hipError_t launch_init_slot(const Slot& slot, Slot* slots, double inner_tol, int max_iter, int max_outer,
                            int precision, hipStream_t s);
hipError_t launch_init(const GridArgs& g, const Slot* slots, int nslots, double inner_tol, int max_iter,
                       int max_outer, int precision, hipStream_t s);
hipError_t launch_setup(const GridArgs& g, const Geometry& geo, const Slot* slots, int nslots,
                        bool write_rho32, hipStream_t s);
// One iteration of the paper's method on all slots (FP64 fields) or one inner
// iteration (FP32 fields).
// HIP events around the launches of one sweep kind inside solves (sweep 0: off);
// the host reads the `used` pairs after the solve and resets `used`.
struct SweepTimer {
    static constexpr int kCap = 256;
    int sweep = 0;
    bool fp32 = false;
    int used = 0;
    hipEvent_t ev[2 * kCap] = {};
};
hipError_t launch_iteration(const GridArgs& g, const Geometry& geo, const Tables& t, const Slot* slots,
                            int nslots, bool fp32, hipStream_t s, SweepTimer* tm = nullptr);
// FP32_REFINE inner iterations in halves: the residual sweep and its decision
// (an evaluation), and the four transform sweeps that apply its update; a
// launch sequence may end on an evaluation and the next start with its update
// (SolveState::upd_due keeps the order).
hipError_t launch_evaluation(const GridArgs& g, const Geometry& geo, const Tables& t, const Slot* slots,
                             int nslots, hipStream_t s, SweepTimer* tm = nullptr);
hipError_t launch_inner_update(const GridArgs& g, const Geometry& geo, const Tables& t, const Slot* slots,
                               int nslots, hipStream_t s, SweepTimer* tm = nullptr);
// One sweep alone (1: P1, 2: P2 and P4, 3: P3, 5: P5), for timing.
hipError_t launch_sweep(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, bool fp32, int which,
                        hipStream_t s);
// poisson_sweeps.hip: one sweep; mode 0 iteration, mode 1 the stand-alone L^+ q
// sweep (FP64).  `share`: fraction of the resident blocks the persistent sweeps
// take.  decide: P1 ends in the iteration's decision (false: timing, the state
// stays as it is).
hipError_t launch_sweep_mode(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, bool fp32, int which,
                             int mode, hipStream_t s, float share = 1.0f, int stage = 1, bool decide = true);
// Sweep number of the launch that does P2, P3 and P4 at once, and the grids that
// have it (k_dht_planes: the same results).
constexpr int kSweepPlanes = 234;
bool planes_fusable(const GridArgs& g, int nslots);
unsigned sweep_groups_x(const GridArgs& g);
// FP32_REFINE: whether rows of this length take the outer residual fused with
// the first inner sweep's residual (one marching column per thread), and that
// sweep alone, ending in its decision unless `decide` is false.
// write = false: the partial sums alone (no r32, no transformed residual).
bool outer_fusable(const GridArgs& g);
hipError_t launch_outer_fused(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, hipStream_t s,
                              float share = 1.0f, bool write = true, bool decide = true);
// FP32_REFINE outer step pieces.
// the FP64 outer residual sweep of rows shorter than 16, not fused, ending in its
// decision unless `decide` is false
hipError_t launch_outer_resid_sweep(const GridArgs& g, const Slot* slots, int nslots, hipStream_t s,
                                    bool decide = true);
// The FP64 outer residual of a refinement step and its decision; where the
// rows allow (*fused), fused with the first inner sweep's residual and, with
// `tail`, followed by the rest of that sweep.  Without `tail` (the final check
// of a solve) fused rows take the residual's sums alone: a solve it does not
// end stays in stage 0, and its next outer residual starts the step.
hipError_t launch_outer_residual(const GridArgs& g, const Geometry& geo, const Tables& t, const Slot* slots,
                                 int nslots, hipStream_t s, bool* fused, bool tail = true);
hipError_t launch_outer_tail(const GridArgs& g, const Geometry& geo, const Tables& t, const Slot* slots,
                             int nslots, hipStream_t s);
hipError_t launch_outer_update(const GridArgs& g, const Geometry& geo, const Slot* slots, int nslots,
                               hipStream_t s);
hipError_t launch_fixup(const GridArgs& g, const Geometry& geo, const Slot* slots, int nslots, hipStream_t s);
// Marks every slot whose solve is not done as done with POISSON_ENOCONV.
hipError_t launch_stop_unfinished(const Slot* slots, int nslots, hipStream_t s);

// Single sweeps for parity checks (one slot).
hipError_t launch_apply(const GridArgs& g, const Geometry& geo, const double* rho, const double* p, double* out,
                        hipStream_t s);
hipError_t launch_residual(const GridArgs& g, const Geometry& geo, const Slot* slot, double* r,
                           hipStream_t s);
// delta (slot.p) = L^+ q (slot.b); fp32: through the FP32 sweeps (q rounded
// to FP32 on load, the result widened from d32 at the end).
hipError_t launch_lap_pinv(const GridArgs& g, const Geometry& geo, const Tables& t, const Slot* slot,
                           hipStream_t s, bool fp32 = false);

// The projection step around the solve (poisson_project.hip): out = div(beta m)
// (rhs == nullptr) or (div(beta m) - rhs) / c_dt; m_d -= c_dt grad_d p.
hipError_t launch_divergence(const GridArgs& g, const double* rho, const double* mx, const double* my,
                             const double* mz, const double* rhs, double c_dt, double* out, hipStream_t s);
hipError_t launch_correct(const GridArgs& g, const double* p, double* mx, double* my, double* mz, double c_dt,
                          hipStream_t s);

// Particles and the grid (poisson_particles.hip): out = P(q) per unit volume
// (ws: particle_workspace_bytes(g, np) bytes of device scratch), out_p =
// I(field)(x_p).  *bad_host = 1 when a position is not finite or too far out
// (then P's output is untouched).  Both return when the work is done.
size_t particle_workspace_bytes(const GridArgs& g, int np);
hipError_t launch_deposit(const GridArgs& g, int np, const double* pos, const double* q, double* out, void* ws,
                          size_t ws_bytes, int* bad_host, hipStream_t s);
hipError_t launch_interpolate(const GridArgs& g, int np, const double* pos, const double* field, double* out,
                              int* bad_dev, int* bad_host, hipStream_t s);

}  // namespace pois
