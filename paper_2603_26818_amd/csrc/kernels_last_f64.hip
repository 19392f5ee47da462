// F64: last-axis passes of the step, the adjoint and the natural layout.
#include "dispatch_impl.hpp"

namespace pfc {
PFC_INSTANTIATE_LAST(double)
}  // namespace pfc
