// batch.hpp -- batched 2D runs: the passes of the single-plan step over many independent instances.
//
// Instances of one shape and one choice of schedules form a group; a pass of a group is one launch,
// blockIdx.y the instance (its entry in the device table) and blockIdx.x the row group or column tile.
// Groups do not depend on each other, so the host runs them on two streams (pfc_api.cpp).  The kernels
// are the single-plan blocks on the same schedules, so every instance is bitwise equal to its own plan.
// Between two steps the x c2r of one and the x r2c of the next are one pass, as in the single plan.
//
// A persistent kernel over all instances, with a grid barrier between passes, took 233 us per step of 48
// FP32 instances (12 each of 128^2 .. 1024^2): 13 us per barrier, one register budget for all sizes (a
// 360-byte call frame), and workgroups that took their items one after the other.  Launches per group and
// pass need no barrier (the next launch waits for the last one's end) and each gets its own tile.
#pragma once

#include "dispatch_impl.hpp"

namespace pfc {

template <typename T, class PL>
__global__ __launch_bounds__(XInvRows<PL>::value *PL::Tp) void batch_x_fwd_kernel(const BatchInst<T> *inst,
                                                                                  const cx<T> *__restrict__ tw,
                                                                                  int lt_shift)
{
    constexpr int ROWS = XInvRows<PL>::value;
    constexpr bool PRE = preload_tw<T, PL>();
    __shared__ cx<T> sh[ROWS * XPitch<T, PL::L, true>::value];
    const BatchInst<T> &in = inst[blockIdx.y];
    XTw<T, PL> pre;
    if constexpr (PRE) load_xtw<T, PL, true>(pre, (int)threadIdx.x % PL::Tp, tw, lt_shift);
    x_r2c_block<T, PL, ROWS, true, true, false, false, PRE>(in.psi, in.scratch, in.n0, tw, lt_shift, blockIdx.x, sh,
                                                            row_pack(PL::L), (int)threadIdx.x, &pre);
}

template <typename T, class PL>
__global__ __launch_bounds__(XInvRows<PL>::value *PL::Tp) void batch_x_inv_kernel(const BatchInst<T> *inst,
                                                                                  const cx<T> *__restrict__ tw,
                                                                                  int lt_shift)
{
    constexpr int ROWS = XInvRows<PL>::value;
    constexpr bool PRE = preload_tw<T, PL>();
    __shared__ cx<T> sh[ROWS * PL::L];
    const BatchInst<T> &in = inst[blockIdx.y];
    XTw<T, PL> pre;
    if constexpr (PRE) load_xtw<T, PL, false>(pre, (int)threadIdx.x % PL::Tp, tw, lt_shift);
    const AdjEpi<T> ea{};
    x_c2r_block<T, PL, ROWS, EPI_PLAIN, false, false, false, false, PRE>(in.scratch, in.psi, in.n0, tw, lt_shift, in.sc, ea,
                                                                         blockIdx.x, sh, row_pack(PL::L),
                                                                         (int)threadIdx.x, &pre);
}

template <typename T, class PLI, class PLF>
__global__ __launch_bounds__((XFused<PLI, PLF, 64>::threads)) void
batch_x_fused_kernel(const BatchInst<T> *inst, const cx<T> *__restrict__ tw, int lt_shift)
{
    __shared__ cx<T> sh[XFused<PLI, PLF, 64>::R * XPitch<T, PLI::L, true>::value];
    const BatchInst<T> &in = inst[blockIdx.y];
    x_c2r_r2c_block<T, PLI, PLF, 64, false, true, true>(in.scratch, in.scratch, in.n0, tw, lt_shift, in.sc, blockIdx.x, sh,
                                                        row_pack(PLI::L));
}

template <typename T, class PL, int WM, bool PF, int G, bool LP>
__global__ __launch_bounds__(WM *PL::Tp) void batch_y_kernel(const BatchInst<T> *inst, int W, int xg,
                                                             const cx<T> *__restrict__ tw, int lt_shift)
{
    constexpr int fold_slots = (LP && PF) ? 2 * PL::L : 0;  // as last_axis_kernel
    __shared__ cx<T> sh[pencil_slot<LP>(PL::L) * WM / G + fold_slots];
    const BatchInst<T> &in = inst[blockIdx.y];
    LastAxisArgs<T> la{};
    la.src = in.scratch;
    la.dst = in.scratch;
    la.state = in.state;
    la.nrows = 1;
    la.M = in.M;
    la.W = W;
    la.tiles_per_row = gridDim.x;
    la.tw = tw;
    la.lt_shift = lt_shift;
    la.mp = in.mp;
    la.pk = row_pack(in.M);
    last_axis_block<T, PL, WM, LA_STEP, PF, ORD_TILE, false, G, LP>(la, xcd_tile_order(blockIdx.x, gridDim.x, xg), sh);
}

// Calls f(std::integral_constant<int, L>) for a length of the batched form: y (32 .. 1024) or x / 2.
template <class F>
hipError_t batch_length(int L, F &&f)
{
    switch (L) {
    case 16: return f(std::integral_constant<int, 16>{});
    case 32: return f(std::integral_constant<int, 32>{});
    case 64: return f(std::integral_constant<int, 64>{});
    case 128: return f(std::integral_constant<int, 128>{});
    case 256: return f(std::integral_constant<int, 256>{});
    case 512: return f(std::integral_constant<int, 512>{});
    case 1024: return f(std::integral_constant<int, 1024>{});
    default: return hipErrorInvalidValue;
    }
}

// Calls f(PL{}, W, PF, G, LP) with the y tile of a group: the single plan's rule over all instances of
// the group, except that FP32 pencils of 256 points and more stay narrow, four together while that leaves
// a workgroup per CU (12 x 1024^2: 50 us; the full tile, 32 elements per thread in two LDS groups, 74 us,
// tiles of two 72 us; 10 steps of 48 x 512^2: 764 against 929 us with full tiles).
template <typename T, class F>
hipError_t batch_y_tile(const BatchGroup &g, F &&f)
{
    return batch_length(g.n0, [&](auto Lc) -> hipError_t {
        constexpr int L = decltype(Lc)::value;
        return with_plan<typename Last2Cands<L>::type>(g.vy, [&](auto plc) -> hipError_t {
            using P0 = decltype(plc);
            using TL = PencilTile<T, L>;
            using PL = SpreadIf<P0, TL::E>;
            using NT = NarrowTile<P0>;
            constexpr std::true_type yes{};
            constexpr std::false_type no{};
            constexpr std::integral_constant<int, 1> one{};
            constexpr std::bool_constant<(P0::Rmax <= 16)> pf{};
            constexpr bool four = sizeof(T) == 4 && NT::W4 > NT::W;
            if constexpr (four)
                if (g.M / NT::W4 * g.count >= kFillTiles) return f(P0{}, std::integral_constant<int, NT::W4>{}, pf, one, yes);
            if (four || cdiv(g.M, TL::W) * g.count < kFillTiles) return f(P0{}, std::integral_constant<int, NT::W>{}, pf, one, yes);
            return f(PL{}, std::integral_constant<int, TL::W>{}, std::bool_constant<TL::PF>{},
                     std::integral_constant<int, TL::G>{}, no);
        });
    });
}

template <typename T>
int64_t batch_y_workgroups(const BatchGroup &g)
{
    int64_t n = 0;
    (void)batch_y_tile<T>(g, [&](auto, auto wc, auto, auto, auto) -> hipError_t {
        n = cdiv(g.M, g.M < wc.value ? g.M : wc.value) * g.count;
        return hipSuccess;
    });
    return n;
}

template <typename T>
hipError_t launch_batch_y(const BatchGroup &g, const BatchInst<T> *table, const cx<T> *tw, int lt_shift, hipStream_t s)
{
    return batch_y_tile<T>(g, [&](auto plc, auto wc, auto pfc, auto gc, auto lpc) -> hipError_t {
        using PL = decltype(plc);
        constexpr int WM = decltype(wc)::value;
        const int W = g.M < WM ? g.M : WM;
        hipLaunchKernelGGL((batch_y_kernel<T, PL, WM, decltype(pfc)::value, decltype(gc)::value, decltype(lpc)::value>),
                           dim3((unsigned)cdiv(g.M, W), (unsigned)g.count), dim3(WM * PL::Tp), 0, s, table + g.first, W,
                           line_group<T>(W), tw, lt_shift);
        return hipGetLastError();
    });
}

template <typename T>
hipError_t launch_batch_x(const BatchGroup &g, int pass, const BatchInst<T> *table, const cx<T> *tw, int lt_shift,
                          hipStream_t s)
{
    return batch_length(g.M, [&](auto Mc) -> hipError_t {
        constexpr int M = decltype(Mc)::value;
        if constexpr (M > 512) {
            return hipErrorInvalidValue;
        } else {
            const BatchInst<T> *inst = table + g.first;
            auto grid = [&](int rows) { return dim3((unsigned)cdiv(g.n0, rows), (unsigned)g.count); };
            if (pass == BATCH_X_FWD)
                return with_plan<typename X2FwdCands<M>::type>(g.vx, [&](auto pf) -> hipError_t {
                    using PL = decltype(pf);
                    constexpr int R = XInvRows<PL>::value;
                    hipLaunchKernelGGL((batch_x_fwd_kernel<T, PL>), grid(R), dim3(R * PL::Tp), 0, s, inst, tw, lt_shift);
                    return hipGetLastError();
                });
            return with_plan<typename X2InvCands<M>::type>(g.vc, [&](auto pi) -> hipError_t {
                using PLI = decltype(pi);
                if (pass == BATCH_X_INV) {
                    constexpr int R = XInvRows<PLI>::value;
                    hipLaunchKernelGGL((batch_x_inv_kernel<T, PLI>), grid(R), dim3(R * PLI::Tp), 0, s, inst, tw, lt_shift);
                    return hipGetLastError();
                }
                return with_plan<typename X2FwdCands<M>::type>(g.vx, [&](auto pf) -> hipError_t {
                    using PLF = decltype(pf);
                    using XF = XFused<PLI, PLF, 64>;
                    static_assert(XF::ok, "both schedules fill one wavefront");
                    hipLaunchKernelGGL((batch_x_fused_kernel<T, PLI, PLF>), grid(XF::R), dim3(XF::threads), 0, s, inst, tw,
                                       lt_shift);
                    return hipGetLastError();
                });
            });
        }
    });
}

}  // namespace pfc
