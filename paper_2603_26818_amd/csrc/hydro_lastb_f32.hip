// F32: last-axis passes of the hydrodynamic step (HYDRO_PSI, HYDRO_VEL).
#include "hydro.hpp"

namespace pfc {
template hipError_t hydro_last_op<float, HYDRO_PSI>(const Geom &, HydroLastArgs<float>, hipStream_t);
template hipError_t hydro_last_op<float, HYDRO_VEL>(const Geom &, HydroLastArgs<float>, hipStream_t);
}  // namespace pfc
