// The y and z sweeps along long lines on FP32 fields.
#include "poisson_columns.hpp"

namespace pois {

template hipError_t launch_cols_y<float, false>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                                int);
template hipError_t launch_z_solve<float, false>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float,
                                                 int);

}  // namespace pois
