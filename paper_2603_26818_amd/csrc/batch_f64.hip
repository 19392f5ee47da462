// FP64: passes of the batched form.
#include "batch.hpp"

namespace pfc {
template int64_t batch_y_workgroups<double>(const BatchGroup &);
template int batch_unit<double>(const BatchGroup &);
template hipError_t launch_batch_y<double>(const BatchGroup *, int, const BatchInst<double> *, const cx<double> *, int,
                                           hipStream_t);
template hipError_t launch_batch_x<double>(const BatchGroup *, int, int, const BatchInst<double> *, const cx<double> *, int,
                                           hipStream_t);
}  // namespace pfc
