// F32: x and y passes of the hydrodynamic step, and its last-axis dispatch.
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
template hipError_t launch_hydro_last<float>(const Geom &, int, const cx<float> *, const cx<float> *, cx<float> *, cx<float> *,
                                        cx<float> *, const HydroArgs &, const cx<float> *, hipStream_t);
template hipError_t launch_hydro_y<float>(const Geom &, cx<float> *, cx<float> *, double, const cx<float> *, hipStream_t);
template hipError_t launch_hydro_x<float>(const Geom &, const HydroFlow<float> &, const cx<float> *, hipStream_t);
template hipError_t launch_hydro_psi_x<float>(const Geom &, const cx<float> *, float *, cx<float> *, const cx<float> *, hipStream_t);
}  // namespace pfc
