// F32: last-axis passes of the hydrodynamic step (HYDRO_DERIV, HYDRO_MU).
#include "hydro.hpp"

namespace pfc {
template hipError_t hydro_last_op<float, HYDRO_DERIV>(const Geom &, HydroLastArgs<float>, hipStream_t);
template hipError_t hydro_last_op<float, HYDRO_MU>(const Geom &, HydroLastArgs<float>, hipStream_t);
}  // namespace pfc
