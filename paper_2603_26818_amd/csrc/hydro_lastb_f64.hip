// F64: last-axis passes of the hydrodynamic step (HYDRO_PSI, HYDRO_VEL).
#include "hydro.hpp"

namespace pfc {
template hipError_t hydro_last_op<double, HYDRO_PSI>(const Geom &, HydroLastArgs<double>, hipStream_t);
template hipError_t hydro_last_op<double, HYDRO_VEL>(const Geom &, HydroLastArgs<double>, hipStream_t);
}  // namespace pfc
