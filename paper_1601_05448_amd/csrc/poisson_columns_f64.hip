// The y and z sweeps along long lines on FP64 fields.
#include "poisson_columns.hpp"

namespace pois {

template hipError_t launch_cols_y<double, false>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                                 int);
template hipError_t launch_z_solve<double, false>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                                  int);

}  // namespace pois
