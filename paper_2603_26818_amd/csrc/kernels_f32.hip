// FP32: passes over grids and modes.
#include "dispatch_impl.hpp"

namespace pfc {
PFC_INSTANTIATE_GRID(float)
}  // namespace pfc
