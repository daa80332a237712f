// The y and z sweeps along short lines, one by one and fused, on FP32 fields.
#include <hip/hip_runtime.h>

// Products and sums are fused within an expression only, as the source says, not
// wherever the optimiser meets them: k_dht_planes and the sweeps that it stands
// for then round alike and give the same bits.  (Long lines stay without it: the
// z sweep of 768 x 768 x 128 spilled, 193 -> 250 us.)
#pragma clang fp contract(on)

#include "poisson_planes.hpp"

namespace pois {

template hipError_t launch_cols_y<float, true>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                               int);
template hipError_t launch_z_solve<float, true>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                                int);
template hipError_t launch_planes<float>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float, int);

}  // namespace pois
