// F32: fused x pass.
#include "dispatch_impl.hpp"

namespace pfc {
PFC_INSTANTIATE_XF(float)
}  // namespace pfc
