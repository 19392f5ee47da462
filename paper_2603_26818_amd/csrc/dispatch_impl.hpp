// dispatch_impl.hpp -- length dispatch of the kernel templates; included once per dtype.
#pragma once

#include "kernels.hpp"
#include "launch.hpp"

namespace pfc {

template <class F>
static hipError_t by_length(int64_t L, F &&f)
{
    switch (L) {
    case 2: return f(std::integral_constant<int, 2>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 8: return f(std::integral_constant<int, 8>{});
    case 16: return f(std::integral_constant<int, 16>{});
    case 32: return f(std::integral_constant<int, 32>{});
    case 64: return f(std::integral_constant<int, 64>{});
    case 128: return f(std::integral_constant<int, 128>{});
    case 256: return f(std::integral_constant<int, 256>{});
    case 512: return f(std::integral_constant<int, 512>{});
    case 1024: return f(std::integral_constant<int, 1024>{});
    case 2048: return f(std::integral_constant<int, 2048>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case 10: return f(std::integral_constant<int, 10>{});
    case 12: return f(std::integral_constant<int, 12>{});
    case 14: return f(std::integral_constant<int, 14>{});
    case 15: return f(std::integral_constant<int, 15>{});
    case 20: return f(std::integral_constant<int, 20>{});
    case 30: return f(std::integral_constant<int, 30>{});
    case 60: return f(std::integral_constant<int, 60>{});
    case 150: return f(std::integral_constant<int, 150>{});
    case 375: return f(std::integral_constant<int, 375>{});
    case 700: return f(std::integral_constant<int, 700>{});
    case 750: return f(std::integral_constant<int, 750>{});
    case 1400: return f(std::integral_constant<int, 1400>{});
    default: return hipErrorInvalidValue;
    }
}

static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Calls f(std::bool_constant<nt>); CAN: whether nt can be true at all, else only one instance is compiled.
template <bool CAN = true, class F>
static hipError_t with_nt(bool nt, F &&f)
{
    if constexpr (CAN)
        if (nt) return f(std::true_type{});
    return f(std::false_type{});
}

// Lengths of by_length that a strided axis (y, last) can have: those of x / 2 include 2 and odd ones.
static constexpr bool axis_length(int L) { return L >= 4 && L % 2 == 0; }

// Every element step of the schedule PL (b Tp + r L / R for its first and last radix) is a
// multiple of the layout's plane block 2^zs, as the last-axis addressing requires (AxisMap, Pack).
template <class PL>
static bool z_steps_ok(int zs)
{
    const int Z = 1 << zs;
    return PL::Tp % Z == 0 && (PL::L / PL::first) % Z == 0 && (PL::L / PL::last) % Z == 0;
}

// Whether blocks of 2^zs z planes suit this geometry's last-axis passes: the step's default z
// schedule and the schedule of the other last-axis passes (state set-up, export, transforms) step
// by multiples of the block.
template <typename T>
bool z_blocks_ok(const Geom &g, int zs)
{
    bool ok = false;
    (void)by_length(g.n0, [&](auto Lc) -> hipError_t {
        constexpr int L = decltype(Lc)::value;
        using TO = TileOf<T, typename ListAt<0, typename ZCandsOf<T, L>::type>::type>;
        using PZ = SpreadIf<typename TO::plan, TO::tile::E>;
        using P0 = SpreadIf<typename LastPlan<L>::type, PencilTile<T, L>::E>;
        ok = z_steps_ok<PZ>(zs) && z_steps_ok<P0>(zs) && z_steps_ok<typename LastPlan<L>::type>(zs);
        return hipSuccess;
    });
    return ok;
}

// Addressing of the middle-axis (3D y) pass: batch = z plane, columns kx, elements y.
static inline AxisMap y_map(const Geom &g)
{
    const Pack pk = pack_of(g);
    return AxisMap{pk.nrows * pk.Mp << pk.zs, pk.Mp << pk.zs, 0, 0, pk.zs, 0, pk.zs, pk.cs};
}
// Addressing of a last-axis c2c pass: one batch, columns row M + kx, elements along the last axis.
static inline AxisMap last_map(const Geom &g)
{
    const Pack pk = pack_of(g);
    return AxisMap{0, pk.e_stride(), pk.Mp << pk.zs, g.M, 0, pk.zs, pk.zs, pk.cs};
}

// Column tiles below which a strided pass takes narrow tiles (NarrowTile in kernels.hpp): one per CU for
// the two transforms of the step and of the adjoint, half of that for a single transform.  Measured per
// step, full tiles then narrow ones: 512^2 FP32 (16 tiles) 17.5 -> 6.5 us for the last-axis pass, 1024 x 32
// x 64 (64 tiles) 82 -> 48 us, 1024 x 64 x 64 (128) 93 -> 69 us; single transforms of 512 x 64 x 64 (128
// tiles) are 5 % slower narrow (hydrodynamic step 2.35 against 2.48 ms), of 512^2 (16) 30 % faster.
constexpr int64_t kFillTiles = 256, kFillTiles1 = 128;

// Calls f with the candidate `variant` of the 2D or the 3D list.
template <class C2, class C3, class F>
static hipError_t with_cands(const Geom &g, int variant, F &&f)
{
    if (g.ndim == 2) return with_plan<C2>(variant, f);
    return with_plan<C3>(variant, f);
}

// Largest even width <= w (w >= 2).
static constexpr int even_width(int w) { return w > 1 ? (w & ~1) : w; }

// Workgroups per 128-byte line for column tiles of W complex values (1 for whole-line tiles).
template <typename T>
__host__ __device__ constexpr int line_group(int W)
{
    const int bytes = W * (int)sizeof(cx<T>);
    return bytes >= 128 ? 1 : 128 / bytes;
}

// Rows per workgroup of the x inverse pass: one wavefront (measured faster than 256 threads; the
// pass's LDS round trips then need no cross-wave barrier), except for mixed-radix rows that fill
// most of a wavefront without dividing it (700 points over 50 threads), which take about 256
// threads as the forward pass does (1400^3 FP32: 8.3 against 9.0 ms).  Over 64 threads a 700-point
// row is one whole wavefront: 7.1 against 8.0 ms with four rows per workgroup; 375-point rows take
// two per wavefront (256 threads measured slower: 1.23 against 1.14 ms).
template <class PL>
struct XInvRows {
    static constexpr int value = (!is_pow2c(PL::L) && PL::Tp > 32 && PL::Tp < 64) ? XRows<PL>::value
                                                                                   : ((64 / PL::Tp) < 1 ? 1 : 64 / PL::Tp);
};

template <typename T>
hipError_t launch_x_r2c(const Geom &g, const T *in, cx<T> *out, bool cube, const cx<T> *tw, hipStream_t s,
                        int variant)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    return by_length(g.M, [&](auto Mc) -> hipError_t {
        constexpr int M = decltype(Mc)::value;
        if constexpr (M > 1024) {
            return hipErrorInvalidValue;
        } else {
            auto run = [&](auto plc, auto cubec) -> hipError_t {
                using PL = decltype(plc);
                constexpr bool CUBE = decltype(cubec)::value;
                // 2D grids (at most 2048 rows): one wavefront per workgroup, which spreads them over more CUs
                if (g.ndim == 2) {
                    constexpr int R1 = XInvRows<PL>::value;
                    hipLaunchKernelGGL((x_r2c_kernel<T, PL, R1, CUBE, is_pow2c(M), false, true>), dim3((unsigned)cdiv(g.xrows, R1)),
                                       dim3(R1 * PL::Tp), 0, s, in, out, g.xrows, tw + g.tw_x, g.lt_shift, pack_of(g));
                    return hipGetLastError();
                }
                constexpr int ROWS = XRows<PL>::value;
                const dim3 grid((unsigned)cdiv(g.xrows, ROWS)), block(ROWS * PL::Tp);
                // non-temporal hints measured faster at M = 256 and slower at M = 1024; mixed-radix
                // rows are not whole lines (their partial lines then reach HBM unmerged).  Padded
                // LDS rows (power-of-two M): 512^3 FP64 x r2c 0.360 against 0.389 ms, FP32 even.
                return with_nt<(M < 1024 && is_pow2c(M))>(g.nt, [&](auto ntc) -> hipError_t {
                    hipLaunchKernelGGL((x_r2c_kernel<T, PL, ROWS, CUBE, is_pow2c(M), decltype(ntc)::value>), grid, block, 0,
                                       s, in, out, g.xrows, tw + g.tw_x, g.lt_shift, pack_of(g));
                    return hipGetLastError();
                });
            };
            using C2 = typename X2FwdCands<M>::type;
            using C3 = typename XFwdCands<M>::type;
            if constexpr (sizeof(T) == 4)
                if (!cube && g.init) return run(typename InitXPlan<M>::type{}, std::false_type{});
            if (!cube)
                return with_cands<PlanList<typename ListAt<0, C2>::type>, PlanList<typename ListAt<0, C3>::type>>(
                    g, 0, [&](auto plc) { return run(plc, std::false_type{}); });
            return with_cands<C2, C3>(g, variant, [&](auto plc) { return run(plc, std::true_type{}); });
        }
    });
}

template <typename T>
hipError_t launch_x_c2r(const Geom &g, const cx<T> *in, T *out, const cx<T> *tw, hipStream_t s, int variant)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    return by_length(g.M, [&](auto Mc) -> hipError_t {
        constexpr int M = decltype(Mc)::value;
        if constexpr (M > 1024) {
            return hipErrorInvalidValue;
        } else {
            return with_cands<typename X2InvCands<M>::type, typename XInvCands<M>::type>(g, variant, [&](auto plc) -> hipError_t {
                using PL = decltype(plc);
                constexpr int ROWS = XInvRows<PL>::value;
                const dim3 grid((unsigned)cdiv(g.xrows, ROWS)), block(ROWS * PL::Tp);
                const T sc = (T)(1.0 / ((double)g.M * (double)g.n0 * (double)g.nrows));
                AdjEpi<T> ea{};
                if (g.ndim == 2) {
                    hipLaunchKernelGGL((x_c2r_kernel<T, PL, ROWS, EPI_PLAIN, false, false, false, true>), grid, block, 0, s, in,
                                       out, g.xrows, tw + g.tw_x, g.lt_shift, sc, ea, pack_of(g));
                    return hipGetLastError();
                }
                // unpadded LDS rows: padded ones measured slower here (512^3 FP32 0.224 against
                // 0.215 ms, FP64 0.419 against 0.396 ms, 2048^3 FP32 18.5 against 18.0 ms)
                return with_nt<is_pow2c(M)>(g.nt, [&](auto ntc) -> hipError_t {
                    hipLaunchKernelGGL((x_c2r_kernel<T, PL, ROWS, EPI_PLAIN, false, false, decltype(ntc)::value>), grid,
                                       block, 0, s, in, out, g.xrows, tw + g.tw_x, g.lt_shift, sc, ea, pack_of(g));
                    return hipGetLastError();
                });
            });
        }
    });
}

// The fused x pass between two steps of the single-plan step (x c2r of one step, the cube, x r2c of
// the next; x_c2r_r2c_kernel), in place on the packed spectrum, on the default x schedules of both
// directions, one wavefront per workgroup.  A geometry has it when both schedules' threads per row
// divide a wavefront and the rows are shorter than 1024 points.  The arithmetic is that of the two
// separate passes, bit for bit.  Measured against the separate passes (whole steps): 512^3 FP32
// 825 against 781 steps/s, FP64 429 against 415, 750^3 186 against 183; at 2048^3 (1024-point rows,
// one row per workgroup) 108.4 against 104.6 ms per step, so rows of 1024 keep the separate passes.
template <class PLI, class PLF>
struct XStepFused {
    static constexpr bool ok = PLI::L == PLF::L && PLI::L < 1024 && PLI::Tp <= 64 && PLF::Tp <= 64 &&
                               64 % PLI::Tp == 0 && 64 % PLF::Tp == 0 && XFused<PLI, PLF, 64>::ok;
};

template <typename T>
bool x_fused_ok(const Geom &g)
{
    if (!layout_ok(g)) return false;
    bool ok = false;
    (void)by_length(g.M, [&](auto Mc) -> hipError_t {
        constexpr int M = decltype(Mc)::value;
        if constexpr (M <= 1024)
            ok = g.ndim == 2 ? XStepFused<typename X2InvPlan<M>::type, typename X2FwdPlan<M>::type>::ok
                             : XStepFused<typename XInvPlan<M>::type, typename XFwdPlan<M>::type>::ok;
        return hipSuccess;
    });
    return ok;
}

template <typename T>
hipError_t launch_x_c2r_r2c(const Geom &g, cx<T> *data, T *real, const cx<T> *tw, hipStream_t s)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    return by_length(g.M, [&](auto Mc) -> hipError_t {
        constexpr int M = decltype(Mc)::value;
        if constexpr (M > 1024) {
            return hipErrorInvalidValue;
        } else {
            auto run = [&](auto pic, auto pfc, auto latc) -> hipError_t {
                using PLI = decltype(pic);
                using PLF = decltype(pfc);
                if constexpr (!XStepFused<PLI, PLF>::ok) {
                    return hipErrorInvalidValue;
                } else {
                    using F = XFused<PLI, PLF, 64>;
                    const dim3 grid((unsigned)cdiv(g.xrows, F::R)), block(F::threads);
                    const T sc = (T)(1.0 / ((double)g.M * (double)g.n0 * (double)g.nrows));
                    // ordinary loads and stores: non-temporal hints (as the separate x passes take them)
                    // measured 1.3 % slower per 512^3 FP32 step, the same in FP64.  Padded LDS rows
                    // (power-of-two M): FP64 steps 438 against 431 steps/s at 512^3, 2768 against 2671
                    // at 256^3; FP32 even.
                    constexpr bool LAT = decltype(latc)::value;
                    if (real)
                        hipLaunchKernelGGL((x_c2r_r2c_kernel<T, PLI, PLF, 64, false, is_pow2c(M), LAT, true>), grid, block, 0, s,
                                           data, real, g.xrows, tw + g.tw_x, g.lt_shift, sc, pack_of(g));
                    else
                        hipLaunchKernelGGL((x_c2r_r2c_kernel<T, PLI, PLF, 64, false, is_pow2c(M), LAT>), grid, block, 0, s, data,
                                           real, g.xrows, tw + g.tw_x, g.lt_shift, sc, pack_of(g));
                    return hipGetLastError();
                }
            };
            if (g.ndim == 2) return run(typename X2InvPlan<M>::type{}, typename X2FwdPlan<M>::type{}, std::true_type{});
            return run(typename XInvPlan<M>::type{}, typename XFwdPlan<M>::type{}, std::false_type{});
        }
    });
}

template <typename T>
hipError_t launch_x_adj_r2c(const Geom &g, cx<T> *data, const cx<T> *nu, const T *psi_n, const T *psi_np1, T c3,
                            double *partial, int64_t slots, bool add, int64_t *nblocks, const cx<T> *tw, hipStream_t s)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    return by_length(g.M, [&](auto Mc) -> hipError_t {
        constexpr int M = decltype(Mc)::value;
        if constexpr (M > 1024) {
            return hipErrorInvalidValue;
        } else {
            auto run = [&](auto pic, auto pfc, auto latc) -> hipError_t {
                using PLI = decltype(pic);
                using PLF = decltype(pfc);
                if constexpr (!XStepFused<PLI, PLF>::ok) {
                    return hipErrorInvalidValue;
                } else {
                    *nblocks = cdiv(g.xrows, XFused<PLI, PLF, 64>::R);
                    if (*nblocks > slots) return hipErrorInvalidValue;
                    const T sc = (T)(1.0 / ((double)g.M * (double)g.n0 * (double)g.nrows));
                    const AdjEpi<T> ea{nu, psi_n, psi_np1, c3, partial, add ? 1 : 0};
                    hipLaunchKernelGGL((x_adj_r2c_kernel<T, PLI, PLF, is_pow2c(M), decltype(latc)::value>),
                                       dim3((unsigned)*nblocks), dim3(XFused<PLI, PLF, 64>::threads), 0, s, data, g.xrows,
                                       tw + g.tw_x, g.lt_shift, sc, ea, pack_of(g));
                    return hipGetLastError();
                }
            };
            if (g.ndim == 2) return run(typename X2InvPlan<M>::type{}, typename X2FwdPlan<M>::type{}, std::true_type{});
            return run(typename XInvPlan<M>::type{}, typename XFwdPlan<M>::type{}, std::false_type{});
        }
    });
}

template <typename T>
hipError_t launch_x_c2r_adjoint(const Geom &g, const cx<T> *mu, const cx<T> *nu, const T *psi_n, const T *psi_np1,
                                T *out, T c3, double *partial, int64_t slots, bool add, int64_t *nblocks, const cx<T> *tw,
                                hipStream_t s)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    return by_length(g.M, [&](auto Mc) -> hipError_t {
        constexpr int M = decltype(Mc)::value;
        if constexpr (M > 1024) {
            return hipErrorInvalidValue;
        } else {
            auto run = [&](auto plc, auto rowsc, auto latc) -> hipError_t {
                using PL = decltype(plc);
                constexpr int ROWS = decltype(rowsc)::value;
                const int64_t nb = cdiv(g.xrows, ROWS);
                *nblocks = nb;
                if (nb > slots) return hipErrorInvalidValue;
                const dim3 grid((unsigned)nb), block(ROWS * PL::Tp);
                const T sc = (T)(1.0 / ((double)g.M * (double)g.n0 * (double)g.nrows));
                AdjEpi<T> ea{nu, psi_n, psi_np1, c3, partial, add ? 1 : 0};
                hipLaunchKernelGGL((x_c2r_kernel<T, PL, ROWS, EPI_ADJOINT, false, false, false, decltype(latc)::value>), grid, block, 0, s, mu, out, g.xrows,
                                   tw + g.tw_x, g.lt_shift, sc, ea, pack_of(g));
                return hipGetLastError();
            };
            using P2 = typename X2InvPlan<M>::type;
            using P3 = typename XInvPlan<M>::type;
            if (g.ndim == 2) return run(P2{}, std::integral_constant<int, XInvRows<P2>::value>{}, std::true_type{});  // as launch_x_r2c
            static_assert(XRows<P3>::value >= kAdjRows3, "the plan counts the partials by it");
            return run(P3{}, std::integral_constant<int, XRows<P3>::value>{}, std::false_type{});
        }
    });
}

template <typename T>
hipError_t launch_y_c2c(const Geom &g, cx<T> *data, int dir, const cx<T> *tw, hipStream_t s, int variant)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    return by_length(g.n1, [&](auto Lc) -> hipError_t {
        constexpr int L = decltype(Lc)::value;
        if constexpr (!axis_length(L)) {
            return hipErrorInvalidValue;
        } else {
            auto run = [&](auto plc) -> hipError_t {
                using TO = TileOf<T, decltype(plc)>;
                using TL = typename TO::tile;
                using PL = SpreadIf<typename TO::plan, TL::E>;
                constexpr int WM = TL::W;
                const int W = (int)(g.M < WM ? g.M : WM);
                const int64_t tiles = cdiv(g.M, W);
                using PN = typename TO::plan;
                constexpr int WN = NarrowTile<PN>::W;
                if constexpr (WN < WM) {
                    if (variant == 0 && tiles * g.n0 < kFillTiles1) {
                        const int w = (int)(g.M < WN ? g.M : WN);
                        const int64_t nt = cdiv(g.M, w);
                        const AxisMap am = y_map(g);
                        if (dir < 0)
                            hipLaunchKernelGGL((axis_c2c_kernel<T, PN, WN, -1, 1, false, 1, true>), dim3((unsigned)(nt * g.n0)),
                                               dim3(WN * PN::Tp), 0, s, data, data, w, g.M, am, nt, tw + g.tw_y, g.lt_shift,
                                               line_group<T>(w));
                        else
                            hipLaunchKernelGGL((axis_c2c_kernel<T, PN, WN, +1, 1, false, 1, true>), dim3((unsigned)(nt * g.n0)),
                                               dim3(WN * PN::Tp), 0, s, data, data, w, g.M, am, nt, tw + g.tw_y, g.lt_shift,
                                               line_group<T>(w));
                        return hipGetLastError();
                    }
                }
                const dim3 grid((unsigned)(tiles * g.n0)), block(WM * PL::Tp);
                // whole-line tiles: whole planes per XCD (xg = 0, see axis_c2c_kernel), except the
                // grouped power-of-two tiles (2048 points), where it measured slower
                const int xg = (line_group<T>(W) == 1 && (TL::G == 1 || !is_pow2c(L))) ? 0 : line_group<T>(W);
                // non-temporal only with whole-line tiles (measured slower on 64-byte tiles)
                return with_nt<line_group<T>(WM) == 1>(g.nt && xg <= 1, [&](auto ntc) -> hipError_t {
                    constexpr bool NT = decltype(ntc)::value;
                    const AxisMap am = y_map(g);
                    if (dir < 0)
                        hipLaunchKernelGGL((axis_c2c_kernel<T, PL, WM, -1, 1, NT, TL::G>), grid, block, 0, s, data,
                                           data, W, g.M, am, tiles, tw + g.tw_y, g.lt_shift, xg);
                    else
                        hipLaunchKernelGGL((axis_c2c_kernel<T, PL, WM, +1, 1, NT, TL::G>), grid, block, 0, s, data,
                                           data, W, g.M, am, tiles, tw + g.tw_y, g.lt_shift, xg);
                    return hipGetLastError();
                });
            };
            // the state set-up: a mixed length's own schedule in the tile of its default candidate
            if constexpr (sizeof(T) == 4 && !is_pow2c(L))
                if (g.init && dir < 0) return run(InitTile<typename ListAt<0, typename AxisCands<L>::type>::type, typename InitAxisPlan<L>::type>{});
            return with_plan<typename AxisCands<L>::type>(variant, run);
        }
    });
}

template <typename T>
hipError_t launch_last_fwd(const Geom &g, const cx<T> *src, cx<T> *dst, const cx<T> *tw, hipStream_t s)
{
    return launch_last_c2c<T>(g, src, dst, -1, tw, s);
}

template <typename T>
hipError_t launch_last_c2c(const Geom &g, const cx<T> *src, cx<T> *dst, int dir, const cx<T> *tw, hipStream_t s)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    return by_length(g.n0, [&](auto Lc) -> hipError_t {
        constexpr int L = decltype(Lc)::value;
        if constexpr (!axis_length(L)) {
            return hipErrorInvalidValue;
        } else {
            constexpr int WM = WMax<T, L>::value;
            const int64_t ncols = g.nrows * g.M;
            const int W = (int)(ncols < WM ? ncols : WM);
            const int64_t tiles = cdiv(ncols, W);
            const AxisMap am = last_map(g);
            auto narrow = [&](auto plc) -> hipError_t {
                using PN = decltype(plc);
                if (!z_steps_ok<PN>(g.zs)) return hipErrorInvalidValue;
                constexpr int WN = NarrowTile<PN>::W;
                const int w = (int)(ncols < WN ? ncols : WN);
                const int64_t nt = cdiv(ncols, w);
                if (dir < 0)
                    hipLaunchKernelGGL((axis_c2c_kernel<T, PN, WN, -1, 1, false, 1, true>), dim3((unsigned)nt),
                                       dim3(WN * PN::Tp), 0, s, src, dst, w, ncols, am, nt, tw + g.tw_last, g.lt_shift,
                                       line_group<T>(w));
                else
                    hipLaunchKernelGGL((axis_c2c_kernel<T, PN, WN, +1, 1, false, 1, true>), dim3((unsigned)nt),
                                       dim3(WN * PN::Tp), 0, s, src, dst, w, ncols, am, nt, tw + g.tw_last, g.lt_shift,
                                       line_group<T>(w));
                return hipGetLastError();
            };
            using PL = typename AxisPlan<L>::type;
            auto forward = [&](auto plc) -> hipError_t {
                using PF = decltype(plc);
                if (!z_steps_ok<PF>(g.zs)) return hipErrorInvalidValue;
                hipLaunchKernelGGL((axis_c2c_kernel<T, PF, WM, -1>), dim3((unsigned)tiles), dim3(WM * PF::Tp), 0, s, src, dst,
                                   W, ncols, am, tiles, tw + g.tw_last, g.lt_shift, 1);
                return hipGetLastError();
            };
            if constexpr (sizeof(T) == 4)
                if (g.init && dir < 0) {
                    using PI = typename InitAxisPlan<L>::type;
                    return tiles < kFillTiles1 ? narrow(PI{}) : forward(PI{});
                }
            if (tiles < kFillTiles1) return g.ndim == 2 ? narrow(typename Last2Plan<L>::type{}) : narrow(PL{});
            if (dir < 0) return forward(PL{});
            if (!z_steps_ok<PL>(g.zs)) return hipErrorInvalidValue;
            const dim3 grid((unsigned)tiles), block(WM * PL::Tp);
            hipLaunchKernelGGL((axis_c2c_kernel<T, PL, WM, +1>), grid, block, 0, s, src, dst, W, ncols, am, tiles,
                                   tw + g.tw_last, g.lt_shift, 1);
            return hipGetLastError();
        }
    });
}

template <typename T>
hipError_t launch_last(const Geom &g, int mode, const cx<T> *src, cx<T> *dst, cx<T> *dst2, cx<T> *state,
                       const ModelParams<T> &mp, const cx<T> *tw, hipStream_t s, int variant)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    return by_length(g.n0, [&](auto Lc) -> hipError_t {
        constexpr int L = decltype(Lc)::value;
        if constexpr (!axis_length(L)) {
            return hipErrorInvalidValue;
        } else {
            constexpr int WM = WMax<T, L>::value;
            LastAxisArgs<T> a{};
            a.src = src;
            a.dst = dst;
            a.dst2 = dst2;
            a.state = state;
            a.nrows = g.nrows;
            a.M = (int)g.M;
            // even tile width: the pair tiles split it between the rows k_y and -k_y
            a.W = even_width(g.M < WM ? (int)g.M : WM);
            a.tiles_per_row = (int)cdiv(g.M, a.W);
            a.tw = tw + g.tw_last;
            a.lt_shift = g.lt_shift;
            a.mp = mp;
            a.pk = pack_of(g);
            a.pk2 = Pack{g.nrows, g.M, 0, 0};  // ADJOINT's nu: plain rows of M
            const int64_t nblocks = (g.nrows == 1) ? a.tiles_per_row : g.nrows * a.tiles_per_row;
            const dim3 grid((unsigned)nblocks);
            using P0 = typename LastPlan<L>::type;
            if (mode != LAST_STEP && !z_steps_ok<P0>(g.zs)) return hipErrorInvalidValue;
            // few tiles: narrow ones (2D grids on the 2D schedules)
            auto narrow_w = [&](auto plc, auto modec, auto wc) -> hipError_t {
                using PN = decltype(plc);
                if (!z_steps_ok<PN>(g.zs)) return hipErrorInvalidValue;
                constexpr int WN = decltype(wc)::value;
                LastAxisArgs<T> b = a;
                b.W = even_width(g.M < WN ? (int)g.M : WN);
                b.tiles_per_row = (int)cdiv(g.M, b.W);
                b.xg = line_group<T>(b.W);
                constexpr bool PF = is_pow2c(L) && PN::Rmax <= 16;  // (mixed lengths as PencilTile)
                hipLaunchKernelGGL((last_axis_kernel<T, PN, WN, decltype(modec)::value, 1, PF, ORD_XCD_ROW, false, 1, true>),
                                   dim3((unsigned)(g.nrows * b.tiles_per_row)), dim3(WN * PN::Tp), 0, s, b);
                return hipGetLastError();
            };
            auto narrow = [&](auto plc, auto modec) -> hipError_t {
                using NT = NarrowTile<decltype(plc)>;
                if constexpr (sizeof(T) == 4 && decltype(modec)::value == LA_STEP && NT::W4 > NT::W)
                    if (g.nrows * (g.M / NT::W4) >= kFillTiles)
                        return narrow_w(plc, modec, std::integral_constant<int, NT::W4>{});
                return narrow_w(plc, modec, std::integral_constant<int, NT::W>{});
            };
            const bool few = nblocks < (mode == LAST_ADJOINT ? kFillTiles : kFillTiles1);
            using P2 = typename Last2Plan<L>::type;
            switch (mode) {
            case LAST_STEP: {
                auto run = [&](auto plc, auto twoc) -> hipError_t {
                    using TO = TileOf<T, decltype(plc)>;
                    using TL = typename TO::tile;
                    using PL = SpreadIf<typename TO::plan, TL::E>;
                    if (!z_steps_ok<PL>(g.zs)) return hipErrorInvalidValue;
                    LastAxisArgs<T> b = a;
                    b.W = even_width(g.M < TL::W ? (int)g.M : TL::W);
                    b.tiles_per_row = (int)cdiv(g.M, b.W);
                    if (variant == 0 && g.nrows * b.tiles_per_row < kFillTiles)
                        return narrow(typename TO::plan{}, std::integral_constant<int, LA_STEP>{});
                    const int64_t nb = (g.nrows == 1) ? b.tiles_per_row : g.nrows * b.tiles_per_row;
                    // (no 2D grid is large enough for non-temporal accesses)
                    constexpr bool CAN = !decltype(twoc)::value && line_group<T>(even_width(TL::W)) == 1;
                    return with_nt<CAN>(g.nt && line_group<T>(b.W) == 1, [&](auto ntc) -> hipError_t {
                        hipLaunchKernelGGL((last_axis_kernel<T, PL, TL::W, LA_STEP, 1, TL::PF, ORD_XCD_ROW,
                                                             decltype(ntc)::value, TL::G>),
                                           dim3((unsigned)nb), dim3(TL::W * PL::Tp), 0, s, b);
                        return hipGetLastError();
                    });
                };
                // 3D: the z candidates (wider tiles at some lengths); 2D: the list the batched
                // kernel shares, so that its instances stay bitwise equal to single plans
                if (g.ndim == 2)
                    return with_plan<typename Last2Cands<L>::type>(variant, [&](auto plc) { return run(plc, std::true_type{}); });
                return with_plan<typename ZCandsOf<T, L>::type>(variant, [&](auto plc) { return run(plc, std::false_type{}); });
            }
            // natural layout (rows of M + 1, not line-aligned): whole rows per XCD, so the lines two
            // tiles share meet in one L2 (measured at 512^3: r2c 403 -> 348 us, c2r 274 -> 262 us)
            case LAST_R2C_NATURAL: {
                // line-aligned output chunks where the geometry allows (3D r2c at 512^3 FP32: 0.734 ->
                // 0.660 ms against the tiles below), else column tiles in whole rows per XCD
                using TL = PencilTile<T, L>;
                constexpr int C = 128 / (int)sizeof(cx<T>);
                if constexpr (TL::W == C && L <= 1024) {  // at 2048 the two rounds' registers would spill
                    if (g.nrows > 1 && (g.nrows * (g.M + 1)) % C == 0 && g.M >= C) {
                        using PL = SpreadIf<P0, TL::E>;
                        if (!z_steps_ok<PL>(g.zs)) return hipErrorInvalidValue;
                        const int64_t nchunks = g.nrows * (g.M + 1) / C;
                        return with_nt(g.nt, [&](auto ntc) -> hipError_t {
                            hipLaunchKernelGGL((r2c_natural_chunk_kernel<T, PL, C, TL::G, decltype(ntc)::value>),
                                               dim3((unsigned)nchunks), dim3(C * PL::Tp), 0, s, src, dst, g.nrows,
                                               (int)g.M, tw + g.tw_last, g.lt_shift, pack_of(g));
                            return hipGetLastError();
                        });
                    }
                }
                if (few) {
                    constexpr std::integral_constant<int, LA_R2C_NATURAL> m{};
                    return g.ndim == 2 ? narrow(P2{}, m) : narrow(P0{}, m);
                }
                hipLaunchKernelGGL((last_axis_kernel<T, P0, WM, LA_R2C_NATURAL, 1, true, ORD_XCD_ROW>), grid,
                                   dim3(WM * P0::Tp), 0, s, a);
                break;
            }
            case LAST_C2R_NATURAL:
                if (few) {
                    constexpr std::integral_constant<int, LA_C2R_NATURAL> m{};
                    return g.ndim == 2 ? narrow(P2{}, m) : narrow(P0{}, m);
                }
                return with_nt<line_group<T>(even_width(WM)) == 1>(g.nt && line_group<T>(a.W) == 1, [&](auto ntc) -> hipError_t {
                    hipLaunchKernelGGL(
                        (last_axis_kernel<T, P0, WM, LA_C2R_NATURAL, 1, true, ORD_XCD_ROW, decltype(ntc)::value>), grid,
                        dim3(WM * P0::Tp), 0, s, a);
                    return hipGetLastError();
                });
            case LAST_ADJOINT:
                if (few) {
                    constexpr std::integral_constant<int, LA_ADJOINT> m{};
                    return g.ndim == 2 ? narrow(P2{}, m) : narrow(P0{}, m);
                }
                hipLaunchKernelGGL((last_axis_kernel<T, P0, WM, LA_ADJOINT>), grid, dim3(WM * P0::Tp), 0, s, a);
                break;
            default: return hipErrorInvalidValue;
            }
            return hipGetLastError();
        }
    });
}

// Threads per row (as a shift) of the passes over modes (for_modes): a quarter of the row's M
// values, so that a thread has its four loads in flight, at most a workgroup's 256.
static inline int row_threads_shift(int64_t M)
{
    int tps = 0;
    while (tps < 8 && (int64_t(4) << tps) < M) ++tps;
    return tps;
}

template <typename T>
hipError_t launch_set_mass(const T *psi, int64_t n, double *partial, cx<T> *state, hipStream_t s)
{
    hipLaunchKernelGGL((sum_kernel<T>), dim3(kReduceBlocks), dim3(256), 0, s, psi, n, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((set_mass_kernel<T>), dim3(1), dim3(256), 0, s, partial, kReduceBlocks, state);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_energy(const Geom &g, const T *psi, const cx<T> *state, const double fk[3], double r, double q1sq,
                         double R1, int model, double dV, double *partial, double *out, hipStream_t s)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    const int64_t ntot = g.n0 * g.nrows * g.nx;
    hipLaunchKernelGGL((energy_kernel<T>), dim3(2 * kReduceBlocks), dim3(256), 0, s, state, psi, g.n0, g.nrows, g.M,
                       row_threads_shift(g.M), fk[0], fk[1], fk[2], r, q1sq, R1, model, kReduceBlocks, partial, pack_of(g));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((energy_final_kernel<T>), dim3(1), dim3(256), 0, s, partial, partial + kReduceBlocks,
                       kReduceBlocks, dV, (double)ntot, state, out);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_export(const Geom &g, const cx<T> *state, cx<T> *out, hipStream_t s)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    const int tps = row_threads_shift(g.M);
    const int64_t blocks = cdiv((g.n0 * g.nrows) << tps, 256);
    hipLaunchKernelGGL((export_kernel<T>), dim3((unsigned)blocks), dim3(256), 0, s, state, out, g.n0, g.nrows, g.M, tps,
                       pack_of(g));
    return hipGetLastError();
}

// Explicit instantiations, in groups: one translation unit per dtype and group, so that they build in
// parallel.
#define PFC_INSTANTIATE_X(T)                                                                                          \
    template hipError_t launch_x_r2c<T>(const Geom &, const T *, cx<T> *, bool, const cx<T> *, hipStream_t, int);     \
    template hipError_t launch_x_c2r<T>(const Geom &, const cx<T> *, T *, const cx<T> *, hipStream_t, int);           \
    template hipError_t launch_x_c2r_adjoint<T>(const Geom &, const cx<T> *, const cx<T> *, const T *, const T *, T *, \
                                                T, double *, int64_t, bool, int64_t *, const cx<T> *, hipStream_t);
#define PFC_INSTANTIATE_XF(T)                                                                                         \
    template hipError_t launch_x_c2r_r2c<T>(const Geom &, cx<T> *, T *, const cx<T> *, hipStream_t);                  \
    template hipError_t launch_x_adj_r2c<T>(const Geom &, cx<T> *, const cx<T> *, const T *, const T *, T, double *,  \
                                            int64_t, bool, int64_t *, const cx<T> *, hipStream_t);                    \
    template bool x_fused_ok<T>(const Geom &);
#define PFC_INSTANTIATE_Y(T)                                                                                          \
    template hipError_t launch_y_c2c<T>(const Geom &, cx<T> *, int, const cx<T> *, hipStream_t, int);                 \
    template hipError_t launch_last_fwd<T>(const Geom &, const cx<T> *, cx<T> *, const cx<T> *, hipStream_t);         \
    template hipError_t launch_last_c2c<T>(const Geom &, const cx<T> *, cx<T> *, int, const cx<T> *, hipStream_t);
#define PFC_INSTANTIATE_LAST(T)                                                                                       \
    template bool z_blocks_ok<T>(const Geom &, int);                                                                  \
    template hipError_t launch_last<T>(const Geom &, int, const cx<T> *, cx<T> *, cx<T> *, cx<T> *,                   \
                                       const ModelParams<T> &, const cx<T> *, hipStream_t, int);
#define PFC_INSTANTIATE_GRID(T)                                                                                       \
    template hipError_t launch_set_mass<T>(const T *, int64_t, double *, cx<T> *, hipStream_t);                       \
    template hipError_t launch_energy<T>(const Geom &, const T *, const cx<T> *, const double *, double, double,      \
                                         double, int, double, double *, double *, hipStream_t);                       \
    template hipError_t launch_export<T>(const Geom &, const cx<T> *, cx<T> *, hipStream_t);

}  // namespace pfc
