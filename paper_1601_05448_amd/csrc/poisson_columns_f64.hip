// The y and z sweeps on FP64 fields.
#include "poisson_columns.hpp"

namespace pois {

template hipError_t launch_cols_y<double>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float, int);
template hipError_t launch_z_solve<double>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                         int);

}  // namespace pois
