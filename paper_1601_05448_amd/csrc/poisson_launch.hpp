// Launch shapes of the persistent sweeps: how many blocks a sweep gets and how
// much LDS a block reserves (poisson_sweeps.hip).
#pragma once

#include "poisson_internal.hpp"

namespace pois {

// Blocks of a persistent sweep: every resident block of the device, shared by
// the slots of the batch, never more than there are line groups.
int persistent_grid(const void* kernel, int threads, unsigned ngroups, int nslots, float share);
// Dynamic LDS bytes a block takes on top of its own so that it has its CU alone
// (a share of at most one half), else 0.
unsigned reserve_lds(const void* kernel, float share);

// A line sweep takes its wide blocks where they make at least this many groups:
// two blocks per CU.
constexpr unsigned kWideGroups = 512;

// One sweep each, MODE as in launch_sweep_mode.  The type selects the FP64 or
// FP32 fields of the slots.
template <typename T>
hipError_t launch_resid(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                        float share, bool decide);
// (Lines of up to kShortLine apart from longer ones: they are compiled with
// k_dht_planes, see poisson_planes_f32.hip.)
constexpr int kShortLine = 64;
template <typename T, bool SHORT>
hipError_t launch_cols_y(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                         float share, int stage);
template <typename T, bool SHORT>
hipError_t launch_z_solve(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                          float share, int stage);
// P2, P3 and P4 as one launch, for grids with planes_fusable.
template <typename T>
hipError_t launch_planes(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                         float share, int stage);
template <typename T>
hipError_t launch_update(const GridArgs& g, const Tables& t, const Slot* slots, int nslots, int mode, hipStream_t s,
                         float share, int stage);

}  // namespace pois
