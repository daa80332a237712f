// The residual sweep P1 on FP64 fields.
#include "poisson_resid.hpp"

namespace pois {

template hipError_t launch_resid<double>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float, bool);

}  // namespace pois
