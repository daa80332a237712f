// The y and z sweeps along short lines, one by one and fused, on FP64 fields.
#include <hip/hip_runtime.h>

// See poisson_planes_f32.hip.  Without it k_dht_planes takes other products into fused
// operations than the sweeps that it stands for; that the bits were equal all the same
// hung on the products' factors being powers of two.  (No time, and no error against
// extended precision, that differs: 32^3 305 and 310 us a solve, 1.51e-15 and 1.52e-15.)
#pragma clang fp contract(on)

#include "poisson_planes.hpp"

namespace pois {

template hipError_t launch_cols_y<double, true>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                                int);
template hipError_t launch_z_solve<double, true>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                                 int);
template hipError_t launch_planes<double>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float, int);

}  // namespace pois
