// batch.hpp -- batched 2D runs: the passes of the single-plan step over many independent instances.
//
// Instances of one shape and one choice of schedules form a group.  A unit is what shares its launches: one
// group, or small groups together (batch_unit).  A pass of a unit is one launch (on tuned schedules one per
// length and schedule); a workgroup takes one row group or column tile of one
// instance, an entry of the device table.  Units do not
// depend on each other, so the host runs them on two streams (pfc_api.cpp).  The kernels are the single-plan
// blocks on the same schedules, so every instance is bitwise equal to its own plan.  Between two steps the
// x c2r of one and the x r2c of the next are one pass, as in the single plan.
//
// A persistent kernel over all instances, with a grid barrier between passes, took 233 us per step of 48
// FP32 instances (12 each of 128^2 .. 1024^2): 13 us per barrier, one register budget for all sizes (a
// 360-byte call frame), and workgroups that took their items one after the other.  Launches per unit and
// pass need no barrier (the next launch waits for the last one's end) and a large group gets its own tile.
#pragma once

#include "dispatch_impl.hpp"

namespace pfc {

// A pass over x: rows per workgroup, LDS slots and the work of workgroup `tile` of an instance, for 64
// threads.  PLI is the inverse schedule, PLF the forward one (each unused in the other's pass).
template <typename T, int PASS, class PLI, class PLF>
struct BatchX;
template <typename T, class PLI, class PL>
struct BatchX<T, BATCH_X_FWD, PLI, PL> {
    static constexpr int rows = XInvRows<PL>::value, threads = rows * PL::Tp;
    static constexpr int slots = rows * XPitch<T, PL::L, true>::value;
    __device__ static __forceinline__ void run(const BatchInst<T> &in, int64_t tile, const cx<T> *__restrict__ tw, int lt_shift,
                                               cx<T> *sh)
    {
        constexpr bool PRE = preload_tw<T, PL>();
        XTw<T, PL> pre;
        if constexpr (PRE) load_xtw<T, PL, true>(pre, (int)threadIdx.x % PL::Tp, tw, lt_shift);
        x_r2c_block<T, PL, rows, true, true, false, false, PRE>(in.psi, in.scratch, in.n0, tw, lt_shift, tile, sh,
                                                                row_pack(PL::L), (int)threadIdx.x, &pre);
    }
};
template <typename T, class PL, class PLF>
struct BatchX<T, BATCH_X_INV, PL, PLF> {
    static constexpr int rows = XInvRows<PL>::value, threads = rows * PL::Tp;
    static constexpr int slots = rows * PL::L;
    __device__ static __forceinline__ void run(const BatchInst<T> &in, int64_t tile, const cx<T> *__restrict__ tw, int lt_shift,
                                               cx<T> *sh)
    {
        constexpr bool PRE = preload_tw<T, PL>();
        XTw<T, PL> pre;
        if constexpr (PRE) load_xtw<T, PL, false>(pre, (int)threadIdx.x % PL::Tp, tw, lt_shift);
        const AdjEpi<T> ea{};
        x_c2r_block<T, PL, rows, EPI_PLAIN, false, false, false, false, PRE>(in.scratch, in.psi, in.n0, tw, lt_shift, in.sc,
                                                                             ea, tile, sh, row_pack(PL::L),
                                                                             (int)threadIdx.x, &pre);
    }
};
template <typename T, class PLI, class PLF>
struct BatchX<T, BATCH_X_FUSED, PLI, PLF> {
    using F = XFused<PLI, PLF, 64>;
    static_assert(F::ok, "both schedules fill one wavefront");
    static constexpr int rows = F::R, threads = F::threads;
    static constexpr int slots = rows * XPitch<T, PLI::L, true>::value;
    __device__ static __forceinline__ void run(const BatchInst<T> &in, int64_t tile, const cx<T> *__restrict__ tw, int lt_shift,
                                               cx<T> *sh)
    {
        x_c2r_r2c_block<T, PLI, PLF, 64, false, true, true>(in.scratch, in.scratch, in.n0, tw, lt_shift, in.sc, tile, sh,
                                                            row_pack(PLI::L));
    }
};

// One group: blockIdx.y the instance, blockIdx.x the row group.
template <typename T, int PASS, class PLI, class PLF>
__global__ __launch_bounds__((BatchX<T, PASS, PLI, PLF>::threads)) void
batch_x_kernel(const BatchInst<T> *inst, const cx<T> *__restrict__ tw, int lt_shift)
{
    __shared__ cx<T> sh[BatchX<T, PASS, PLI, PLF>::slots];
    BatchX<T, PASS, PLI, PLF>::run(inst[blockIdx.y], blockIdx.x, tw, lt_shift, sh);
}

// Tile `bid` of `tiles` of the y pass of an instance.
template <typename T, class PL, int WM, bool PF, int G, bool LP>
__device__ __forceinline__ void batch_y_block(const BatchInst<T> &in, int W, int64_t bid, int tiles, int xg,
                                              const cx<T> *__restrict__ tw, int lt_shift, cx<T> *sh)
{
    LastAxisArgs<T> la{};
    la.src = in.scratch;
    la.dst = in.scratch;
    la.state = in.state;
    la.nrows = 1;
    la.M = in.M;
    la.W = W;
    la.tiles_per_row = tiles;
    la.tw = tw;
    la.lt_shift = lt_shift;
    la.mp = in.mp;
    la.pk = row_pack(in.M);
    last_axis_block<T, PL, WM, LA_STEP, PF, ORD_TILE, false, G, LP>(la, xcd_tile_order(bid, tiles, xg), sh);
}
template <class PL, int WM, bool PF, int G, bool LP>
constexpr int batch_y_slots()  // as last_axis_kernel
{
    return pencil_slot<LP>(PL::L) * WM / G + ((LP && PF) ? 2 * PL::L : 0);
}

template <typename T, class PL, int WM, bool PF, int G, bool LP>
__global__ __launch_bounds__(WM *PL::Tp) void batch_y_kernel(const BatchInst<T> *inst, int W, int xg,
                                                             const cx<T> *__restrict__ tw, int lt_shift)
{
    __shared__ cx<T> sh[batch_y_slots<PL, WM, PF, G, LP>()];
    batch_y_block<T, PL, WM, PF, G, LP>(inst[blockIdx.y], W, blockIdx.x, (int)gridDim.x, xg, tw, lt_shift, sh);
}

// Several groups in one launch.  The workgroup's group is the last one that begins at or before it; all counts
// are powers of two.
struct BatchTiles {
    struct Group {
        int begin;  // its first workgroup
        int first;  // its first instance
        int shift;  // log2 of the workgroups per instance
        int len;    // length of the pass: y, or x / 2
    } g[kBatchUnitGroups];
    int n;
};
struct BatchPlace {
    int inst, tile, tiles, len;
};
__device__ __forceinline__ BatchPlace batch_place(const BatchTiles &b)
{
    const int lane = threadIdx.x & 63, bid = (int)blockIdx.x;
    const bool begun = lane < b.n && b.g[lane].begin <= bid;
    const int i = __builtin_amdgcn_readfirstlane(__popcll(__ballot(begun)) - 1);
    const int w = bid - b.g[i].begin, sh = b.g[i].shift;
    return {b.g[i].first + (w >> sh), w & ((1 << sh) - 1), 1 << sh, b.g[i].len};
}

constexpr int kBatchMinX = 4, kBatchMaxX = 9;  // log2 of x / 2
template <int M>
using BatchXI = typename X2InvPlan<M>::type;
template <int M>
using BatchXF = typename X2FwdPlan<M>::type;
template <typename T, int PASS, int K = kBatchMinX>
constexpr int batch_x_slots()
{
    if constexpr (K > kBatchMaxX) {
        return 0;
    } else {
        constexpr int M = 1 << K, here = BatchX<T, PASS, BatchXI<M>, BatchXF<M>>::slots, rest = batch_x_slots<T, PASS, K + 1>();
        return here > rest ? here : rest;
    }
}
template <typename T, int PASS>
__global__ __launch_bounds__(64) void batch_x_many_kernel(BatchTiles b, const BatchInst<T> *table,
                                                          const cx<T> *__restrict__ tw, int lt_shift)
{
    __shared__ cx<T> sh[batch_x_slots<T, PASS>()];
    const BatchPlace w = batch_place(b);
    const BatchInst<T> &in = table[w.inst];
    static_for<kBatchMinX, kBatchMaxX + 1>([&](auto kc) {
        constexpr int M = 1 << decltype(kc)::value;
        using X = BatchX<T, PASS, BatchXI<M>, BatchXF<M>>;
        static_assert(X::threads == 64, "every length takes one wavefront");
        if (w.len == M) X::run(in, w.tile, tw, lt_shift, sh);  // uniform per workgroup
    });
}

// y lengths 2^K0 .. 2^K1, which take narrow tiles of one number of threads.
template <int L>
using BatchY = typename Last2Plan<L>::type;
template <int K, int K1>
constexpr int batch_y_many_slots()
{
    if constexpr (K > K1) {
        return 0;
    } else {
        using PL = BatchY<(1 << K)>;
        constexpr int here = batch_y_slots<PL, NarrowTile<PL>::W, true, 1, true>(), rest = batch_y_many_slots<K + 1, K1>();
        return here > rest ? here : rest;
    }
}
template <int K>
constexpr int batch_y_threads() { return NarrowTile<BatchY<(1 << K)>>::W * BatchY<(1 << K)>::Tp; }
template <typename T, int K0, int K1>
__global__ __launch_bounds__(batch_y_threads<K0>()) void batch_y_many_kernel(BatchTiles b, const BatchInst<T> *table,
                                                                             const cx<T> *__restrict__ tw, int lt_shift)
{
    __shared__ cx<T> sh[batch_y_many_slots<K0, K1>()];
    const BatchPlace w = batch_place(b);
    const BatchInst<T> &in = table[w.inst];
    static_for<K0, K1 + 1>([&](auto kc) {
        constexpr int L = 1 << decltype(kc)::value;
        using PL = BatchY<L>;
        constexpr int W = NarrowTile<PL>::W;
        static_assert(W * PL::Tp == batch_y_threads<K0>() && PL::Rmax <= 16, "one tile form per class");
        if (w.len == L)  // uniform per workgroup
            batch_y_block<T, PL, W, true, 1, true>(in, W, w.tile, w.tiles, line_group<T>(W), tw, lt_shift, sh);
    });
}

// The same for groups on tuned schedules: one length and schedule, any number of shapes.
template <typename T, int PASS, class PLI, class PLF>
__global__ __launch_bounds__((BatchX<T, PASS, PLI, PLF>::threads)) void
batch_x_set_kernel(BatchTiles b, const BatchInst<T> *table, const cx<T> *__restrict__ tw, int lt_shift)
{
    __shared__ cx<T> sh[BatchX<T, PASS, PLI, PLF>::slots];
    const BatchPlace w = batch_place(b);
    BatchX<T, PASS, PLI, PLF>::run(table[w.inst], w.tile, tw, lt_shift, sh);
}
template <typename T, class PL>
__global__ __launch_bounds__(NarrowTile<PL>::W *PL::Tp) void batch_y_set_kernel(BatchTiles b, const BatchInst<T> *table,
                                                                                const cx<T> *__restrict__ tw, int lt_shift)
{
    constexpr int W = NarrowTile<PL>::W;
    constexpr bool PF = PL::Rmax <= 16;
    __shared__ cx<T> sh[batch_y_slots<PL, W, PF, 1, true>()];
    const BatchPlace w = batch_place(b);
    batch_y_block<T, PL, W, PF, 1, true>(table[w.inst], W, w.tile, w.tiles, line_group<T>(W), tw, lt_shift, sh);
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
        constexpr int L = decltype(Lc)::value < 32 ? 32 : decltype(Lc)::value;  // (16 only as x / 2)
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

inline bool batch_tuned(const BatchGroup &g) { return g.vx != 0 || g.vy != 0 || g.vc != 0; }

// The unit that a group shares its launches in, or 0.  A group is small where it takes narrow tiles.  Small
// groups on the default schedules run together by class of y lengths (up to 256, 512, 1024 points), whose
// narrow tiles are of one form; those on tuned schedules are one unit, with a launch per length and schedule.
// Apart, every shape costs two launches of 5 to 9 us per step, one after the other.  50 steps, us per step,
// in the persistent kernel, apart, together: all 36 shapes, one instance each, FP32 122, 237, 53, FP64 204,
// 289, 72, four of each FP32 254, 300, 157, FP64 660, 422, 256; 9 shapes up to 128 x 128, 16 of each, FP32
// 70, 59, 20; 4 squares of 128 .. 1024, 12 of each, FP32 230, 106, 106.
template <typename T>
int batch_unit(const BatchGroup &g)
{
    bool narrow = false;
    (void)batch_y_tile<T>(g, [&](auto plc, auto wc, auto, auto, auto lpc) -> hipError_t {
        narrow = decltype(lpc)::value && wc.value == NarrowTile<decltype(plc)>::W;
        return hipSuccess;
    });
    return !narrow ? 0 : batch_tuned(g) ? 1 : g.n0 <= 256 ? 256 : g.n0;
}

// Calls f(groups, number) for the groups of each value of key(group), at most kBatchUnitGroups at a time.
template <class Key, class F>
hipError_t batch_by_key(const BatchGroup *g, int ng, Key &&key, F &&f)
{
    if (ng > kBatchMaxInstHost) return hipErrorInvalidValue;
    bool done[kBatchMaxInstHost] = {};
    for (int i = 0; i < ng; ++i) {
        if (done[i]) continue;
        BatchGroup sub[kBatchUnitGroups];
        int n = 0;
        for (int j = i; j < ng && n < kBatchUnitGroups; ++j)
            if (!done[j] && key(g[j]) == key(g[i])) {
                sub[n++] = g[j];
                done[j] = true;
            }
        const hipError_t e = f((const BatchGroup *)sub, n);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The launch's table for groups of `tiles(g)` workgroups per instance and pass length `len(g)`, and its
// workgroups in *total; false where the groups are not what the kernels take.
template <class Tiles, class Len>
bool batch_tiles(const BatchGroup *g, int ng, Tiles &&tiles, Len &&len, BatchTiles *b, int64_t *total)
{
    if (ng > kBatchUnitGroups) return false;
    *total = 0;
    for (int i = 0; i < ng; ++i) {
        const int64_t n = tiles(g[i]);
        if (n < 1 || (n & (n - 1)) != 0) return false;
        int shift = 0;
        while ((int64_t(1) << shift) < n) ++shift;
        b->g[i] = {(int)*total, g[i].first, shift, len(g[i])};
        *total += n * g[i].count;
    }
    b->n = ng;
    return true;
}

template <typename T>
hipError_t launch_batch_y(const BatchGroup *g, int ng, const BatchInst<T> *table, const cx<T> *tw, int lt_shift, hipStream_t s)
{
    if (ng == 1)
        return batch_y_tile<T>(*g, [&](auto plc, auto wc, auto pfc, auto gc, auto lpc) -> hipError_t {
            using PL = decltype(plc);
            constexpr int WM = decltype(wc)::value;
            const int W = g->M < WM ? g->M : WM;
            hipLaunchKernelGGL((batch_y_kernel<T, PL, WM, decltype(pfc)::value, decltype(gc)::value, decltype(lpc)::value>),
                               dim3((unsigned)cdiv(g->M, W), (unsigned)g->count), dim3(WM * PL::Tp), 0, s, table + g->first, W,
                               line_group<T>(W), tw, lt_shift);
            return hipGetLastError();
        });
    if (batch_tuned(*g))
        return batch_by_key(
            g, ng, [](const BatchGroup &q) { return q.n0 * 8 + q.vy; },
            [&](const BatchGroup *sub, int n) -> hipError_t {
                if (n == 1) return launch_batch_y<T>(sub, 1, table, tw, lt_shift, s);
                return batch_length(sub->n0, [&](auto Lc) -> hipError_t {
                    constexpr int L = decltype(Lc)::value < 32 ? 32 : decltype(Lc)::value;
                    return with_plan<typename Last2Cands<L>::type>(sub->vy, [&](auto plc) -> hipError_t {
                        using PL = decltype(plc);
                        constexpr int W = NarrowTile<PL>::W;
                        BatchTiles b{};
                        int64_t total = 0;
                        if (!batch_tiles(sub, n, [](const BatchGroup &q) -> int64_t { return q.M / W; },
                                         [](const BatchGroup &q) { return q.n0; }, &b, &total))
                            return hipErrorInvalidValue;
                        hipLaunchKernelGGL((batch_y_set_kernel<T, PL>), dim3((unsigned)total), dim3(W * PL::Tp), 0, s, b, table,
                                           tw, lt_shift);
                        return hipGetLastError();
                    });
                });
            });
    auto run = [&](auto k0, auto k1) -> hipError_t {
        constexpr int K0 = decltype(k0)::value, K1 = decltype(k1)::value;
        BatchTiles b{};
        int64_t total = 0;
        const bool ok = batch_tiles(
            g, ng,
            [&](const BatchGroup &q) -> int64_t {
                int64_t n = 0;
                (void)batch_length(q.n0, [&](auto Lc) -> hipError_t {
                    constexpr int L = decltype(Lc)::value;
                    if constexpr (L >= (1 << K0) && L <= (1 << K1)) n = q.M / NarrowTile<BatchY<L>>::W;
                    return hipSuccess;
                });
                return n;
            },
            [](const BatchGroup &q) { return q.n0; }, &b, &total);
        if (!ok) return hipErrorInvalidValue;
        hipLaunchKernelGGL((batch_y_many_kernel<T, K0, K1>), dim3((unsigned)total), dim3(batch_y_threads<K0>()), 0, s, b, table,
                           tw, lt_shift);
        return hipGetLastError();
    };
    constexpr std::integral_constant<int, 5> k5{};
    constexpr std::integral_constant<int, 8> k8{};
    constexpr std::integral_constant<int, 9> k9{};
    constexpr std::integral_constant<int, 10> k10{};
    return g->n0 <= 256 ? run(k5, k8) : g->n0 == 512 ? run(k9, k9) : run(k10, k10);
}

// Calls f(std::integral_constant<int, pass>, PLI{}, PLF{}) with a group's x schedules (of the passes that have
// one of the two, it is given twice).
template <typename T, class F>
hipError_t batch_x_schedule(const BatchGroup &g, int pass, F &&f)
{
    return batch_length(g.M, [&](auto Mc) -> hipError_t {
        constexpr int M = decltype(Mc)::value;
        if constexpr (M > 512) {
            return hipErrorInvalidValue;
        } else {
            if (pass == BATCH_X_FWD)
                return with_plan<typename X2FwdCands<M>::type>(
                    g.vx, [&](auto pf) { return f(std::integral_constant<int, BATCH_X_FWD>{}, pf, pf); });
            return with_plan<typename X2InvCands<M>::type>(g.vc, [&](auto pi) -> hipError_t {
                if (pass == BATCH_X_INV) return f(std::integral_constant<int, BATCH_X_INV>{}, pi, pi);
                return with_plan<typename X2FwdCands<M>::type>(
                    g.vx, [&](auto pf) { return f(std::integral_constant<int, BATCH_X_FUSED>{}, pi, pf); });
            });
        }
    });
}

template <typename T>
hipError_t launch_batch_x(const BatchGroup *g, int ng, int pass, const BatchInst<T> *table, const cx<T> *tw, int lt_shift,
                          hipStream_t s)
{
    if (ng > 1 && batch_tuned(*g))
        return batch_by_key(
            g, ng,
            [&](const BatchGroup &q) { return (q.M * 8 + (pass == BATCH_X_INV ? 0 : q.vx)) * 8 + (pass == BATCH_X_FWD ? 0 : q.vc); },
            [&](const BatchGroup *sub, int n) -> hipError_t {
                if (n == 1) return launch_batch_x<T>(sub, 1, pass, table, tw, lt_shift, s);
                return batch_x_schedule<T>(*sub, pass, [&](auto passc, auto pic, auto pfc) -> hipError_t {
                    using PLI = decltype(pic);
                    using PLF = decltype(pfc);
                    constexpr int PASS = decltype(passc)::value;
                    using X = BatchX<T, PASS, PLI, PLF>;
                    BatchTiles b{};
                    int64_t total = 0;
                    if (!batch_tiles(sub, n, [](const BatchGroup &q) -> int64_t { return cdiv(q.n0, X::rows); },
                                     [](const BatchGroup &q) { return q.M; }, &b, &total))
                        return hipErrorInvalidValue;
                    hipLaunchKernelGGL((batch_x_set_kernel<T, PASS, PLI, PLF>), dim3((unsigned)total), dim3(X::threads), 0, s, b,
                                       table, tw, lt_shift);
                    return hipGetLastError();
                });
            });
    if (ng > 1) {
        auto run = [&](auto passc) -> hipError_t {
            constexpr int PASS = decltype(passc)::value;
            BatchTiles b{};
            int64_t total = 0;
            const bool ok = batch_tiles(
                g, ng,
                [&](const BatchGroup &q) -> int64_t {
                    int64_t n = 0;
                    (void)batch_length(q.M, [&](auto Mc) -> hipError_t {
                        constexpr int M = decltype(Mc)::value;
                        if constexpr (M <= (1 << kBatchMaxX)) n = cdiv(q.n0, BatchX<T, PASS, BatchXI<M>, BatchXF<M>>::rows);
                        return hipSuccess;
                    });
                    return n;
                },
                [](const BatchGroup &q) { return q.M; }, &b, &total);
            if (!ok) return hipErrorInvalidValue;
            hipLaunchKernelGGL((batch_x_many_kernel<T, PASS>), dim3((unsigned)total), dim3(64), 0, s, b, table, tw, lt_shift);
            return hipGetLastError();
        };
        if (pass == BATCH_X_FWD) return run(std::integral_constant<int, BATCH_X_FWD>{});
        if (pass == BATCH_X_INV) return run(std::integral_constant<int, BATCH_X_INV>{});
        return run(std::integral_constant<int, BATCH_X_FUSED>{});
    }
    return batch_x_schedule<T>(*g, pass, [&](auto passc, auto pic, auto pfc) -> hipError_t {
        using PLI = decltype(pic);
        using PLF = decltype(pfc);
        constexpr int PASS = decltype(passc)::value;
        using X = BatchX<T, PASS, PLI, PLF>;
        hipLaunchKernelGGL((batch_x_kernel<T, PASS, PLI, PLF>), dim3((unsigned)cdiv(g->n0, X::rows), (unsigned)g->count),
                           dim3(X::threads), 0, s, table + g->first, tw, lt_shift);
        return hipGetLastError();
    });
}

}  // namespace pfc
