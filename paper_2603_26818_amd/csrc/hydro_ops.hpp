// hydro_ops.hpp -- the last-axis operations live in translation units of their own (hydro_last*.hip).
#pragma once

#include "hydro.hpp"

namespace pfc {
#define PFC_HYDRO_EXTERN(T)                                                                                \
    extern template hipError_t hydro_last_op<T, HYDRO_DERIV>(const Geom &, HydroLastArgs<T>, hipStream_t); \
    extern template hipError_t hydro_last_op<T, HYDRO_MU>(const Geom &, HydroLastArgs<T>, hipStream_t);    \
    extern template hipError_t hydro_last_op<T, HYDRO_PSI>(const Geom &, HydroLastArgs<T>, hipStream_t);   \
    extern template hipError_t hydro_last_op<T, HYDRO_VEL>(const Geom &, HydroLastArgs<T>, hipStream_t);
PFC_HYDRO_EXTERN(float)
PFC_HYDRO_EXTERN(double)
#undef PFC_HYDRO_EXTERN
}  // namespace pfc
