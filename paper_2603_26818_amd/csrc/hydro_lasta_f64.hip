// F64: last-axis passes of the hydrodynamic step (HYDRO_DERIV, HYDRO_MU).
#include "hydro.hpp"

namespace pfc {
template hipError_t hydro_last_op<double, HYDRO_DERIV>(const Geom &, HydroLastArgs<double>, hipStream_t);
template hipError_t hydro_last_op<double, HYDRO_MU>(const Geom &, HydroLastArgs<double>, hipStream_t);
}  // namespace pfc
