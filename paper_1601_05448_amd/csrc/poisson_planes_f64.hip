// The y and z sweeps along short lines, one by one and fused, on FP64 fields.
#include "poisson_planes.hpp"

namespace pois {

template hipError_t launch_cols_y<double, true>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                                int);
template hipError_t launch_z_solve<double, true>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                                 int);
template hipError_t launch_planes<double>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float, int);

}  // namespace pois
