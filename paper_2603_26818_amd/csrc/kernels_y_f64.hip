// F64: y and last-axis transforms.
#include "dispatch_impl.hpp"

namespace pfc {
PFC_INSTANTIATE_Y(double)
}  // namespace pfc
