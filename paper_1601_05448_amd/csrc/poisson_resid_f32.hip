// The residual sweep P1 on FP32 fields.
#include "poisson_resid.hpp"

namespace pois {

template hipError_t launch_resid<float>(const GridArgs&, const Tables&, const Slot*, int, int, hipStream_t, float, bool);

}  // namespace pois
