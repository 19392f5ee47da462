// F64: separate x passes.
#include "dispatch_impl.hpp"

namespace pfc {
PFC_INSTANTIATE_X(double)
}  // namespace pfc
