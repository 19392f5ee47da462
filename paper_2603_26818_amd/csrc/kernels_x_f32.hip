// F32: separate x passes.
#include "dispatch_impl.hpp"

namespace pfc {
PFC_INSTANTIATE_X(float)
}  // namespace pfc
