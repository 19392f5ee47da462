// FP32: passes of the batched form; its candidate counts.
#include "batch.hpp"

namespace pfc {
template int64_t batch_y_workgroups<float>(const BatchGroup &);
template int batch_unit<float>(const BatchGroup &);
template hipError_t launch_batch_y<float>(const BatchGroup *, int, const BatchInst<float> *, const cx<float> *, int, hipStream_t);
template hipError_t launch_batch_x<float>(const BatchGroup *, int, int, const BatchInst<float> *, const cx<float> *, int,
                                        hipStream_t);

int batch_candidates(int n0, int M, int pass)
{
    int n = 0;
    (void)batch_length(pass == 1 ? n0 : M, [&](auto Lc) -> hipError_t {
        constexpr int L = decltype(Lc)::value;
        n = pass == 1 ? Last2Cands<L>::type::size : pass == 0 ? X2FwdCands<L>::type::size : X2InvCands<L>::type::size;
        return hipSuccess;
    });
    return n;
}
}  // namespace pfc
