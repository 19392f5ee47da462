// F64: x and y passes of the hydrodynamic step, and its last-axis dispatch.
#include "hydro.hpp"
#include "hydro_ops.hpp"

namespace pfc {
template <typename T>
hipError_t launch_hydro_last(const Geom &g, int op, const cx<T> *a, const cx<T> *b, cx<T> *s, cx<T> *o0, cx<T> *o1,
                             const HydroArgs &h, const cx<T> *tw, hipStream_t st)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    const HydroLastArgs<T> r = hydro_last_args<T>(g, a, b, s, o0, o1, h, tw);
    switch (op) {
    case HYDRO_DERIV: return hydro_last_op<T, HYDRO_DERIV>(g, r, st);
    case HYDRO_MU: return hydro_last_op<T, HYDRO_MU>(g, r, st);
    case HYDRO_PSI: return hydro_last_op<T, HYDRO_PSI>(g, r, st);
    case HYDRO_VEL: return hydro_last_op<T, HYDRO_VEL>(g, r, st);
    default: return hipErrorInvalidValue;
    }
}
template hipError_t launch_hydro_last<double>(const Geom &, int, const cx<double> *, const cx<double> *, cx<double> *, cx<double> *,
                                        cx<double> *, const HydroArgs &, const cx<double> *, hipStream_t);
template hipError_t launch_hydro_y<double>(const Geom &, cx<double> *, cx<double> *, double, const cx<double> *, hipStream_t);
template hipError_t launch_hydro_x<double>(const Geom &, const HydroFlow<double> &, const cx<double> *, hipStream_t);
template hipError_t launch_hydro_psi_x<double>(const Geom &, const cx<double> *, double *, cx<double> *, const cx<double> *, hipStream_t);
}  // namespace pfc
