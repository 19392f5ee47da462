// hydro.hpp -- kernels of the hydrodynamic PFC step (arxiv 2603.26818, Eq. (5)-(6), Listing 2).
//
// The step is bound by HBM traffic (16 transforms of field-sized arrays), so its kernels merge what
// reads the same data:
//   last axis: the forward transforms, the spectral update of a field and the inverse transform in one
//     kernel; mu (or the state) gives its plain inverse transform and that of its last-axis derivative
//     from one read.  i k_y and i k_x commute with the other axes' transforms, so the y and x
//     derivatives share the plain one and are applied in the y and x passes;
//   y: the plain inverse and that of i k_y from one read;
//   x: the fields of a row, their products with real fields and the row transform of the result.
// Per 3D step 79 reads or writes of a field's size (75 where the spectrum of psi^3 is kept for the next
// step), where separate passes for every transform and update make 120.  512^3 FP32: 12.9 ms per step
// separate (297 us per x product pass, 303 us per derivative, 385-484 us per update and 200 us for each
// transform pass beside it); now 9.3 ms: last axis 335 us (gradient, 3 field passes, 4.8 TB/s), 718 us
// (density, 5, 3.7 TB/s), 592 us (mu, 4) and 512 us (velocity, 4), y pair 289 us (3, 5.6 TB/s), x 1085 us
// (advection, 7), 418 us (one force, 3) and 438 us (density, 3).
#pragma once

#include "dispatch_impl.hpp"

namespace pfc {

__device__ __forceinline__ double hy_corr(const HydroArgs &h, double q)
{
    const double a = (1.0 - q) * (1.0 - q);
    if (h.model == 0) return a;
    const double b = h.q1sq - q;
    return a * (b * b + h.R1);
}

// The update of one mode for its q in FP64, with real coefficients (so it maps Hermitian planes to
// Hermitian planes):
//   HYDRO_PSI: S <- (S - dt q nl N - dt B) / (1 + dt q (r + L(q)))    (o = S, a = N, b = B)
//   HYDRO_MU:  A <- nl A + (r + L(q)) S                                 (o = A, a = S)
//   HYDRO_VEL: V <- (V - c G(q) B) / (1 + c Gamma q), G = exp(-a0^2 q/2) (o = V, a = B)
template <int OP>
__device__ __forceinline__ void hy_mode(const HydroArgs &h, double q, double o[2], const double a[2], const double b[2])
{
    if constexpr (OP == HYDRO_PSI) {
        const double den = 1.0 + h.dt * q * (h.r + hy_corr(h, q)), f = -h.dt * q * h.nl;
        for (int c = 0; c < 2; ++c) o[c] = (o[c] + f * a[c] - h.dt * b[c]) / den;
    } else if constexpr (OP == HYDRO_MU) {
        const double m = h.r + hy_corr(h, q);
        for (int c = 0; c < 2; ++c) o[c] = h.nl * o[c] + m * a[c];
    } else {
        const double g = h.c * exp(-0.5 * h.a0 * h.a0 * q), den = 1.0 + h.c * h.gamma * q;
        for (int c = 0; c < 2; ++c) o[c] = (o[c] - g * a[c]) / den;
    }
}

template <typename T>
struct HydroLastArgs {
    const cx<T> *a, *b;
    cx<T> *s, *o0, *o1;  // launch_hydro_last
    int64_t nrows;
    int M, W, tiles_per_row, xg;
    const cx<T> *tw;
    int lt_shift;
    HydroArgs h;
    Pack pk;
};

// Operands that the folded column exchanges through LDS: mirror values of two arrays, of three in the
// FP32 density update (FP64 combines S - dt B first, which is exact enough only there).
template <typename T, int OP>
constexpr int hy_fold_arrays() { return OP == HYDRO_DERIV ? 0 : (OP == HYDRO_PSI && sizeof(T) == 4) ? 3 : 2; }
// LDS slots: the exchange tile, or the folded pencils (two per pair tile) that reuse it
template <typename T, class PL, int WMAX, int OP, bool LP>
constexpr int hy_lds()
{
    constexpr int tile = pencil_slot<LP>(PL::L) * WMAX, fold = 2 * PL::L * hy_fold_arrays<T, OP>();
    return tile > fold ? tile : fold;
}

// Last-axis pass (tiles and pairs as last_axis_block).  A workgroup holds all of its pencils' elements
// before it stores, so o0 may be one of the inputs.  SHORT: 3D rows of one tile, in the order of la_pair_order.
template <typename T, class PL, int WMAX, int OP, bool NT, bool LP, bool SHORT = false>
__global__ __launch_bounds__(WMAX *PL::Tp) void hydro_last_kernel(HydroLastArgs<T> a)
{
    constexpr int L = PL::L, Tp = PL::Tp, Rmax = PL::Rmax, R0 = PL::first, Rl = PL::last;
    using PR = typename PL::Reverse;
    constexpr int Rf = PR::last;
    // the state is loaded ahead of the forward transforms where its registers fit beside theirs
    constexpr bool PF = OP != HYDRO_DERIV && (int)sizeof(T) * Rmax <= (OP == HYDRO_PSI ? 32 : 64);
    __shared__ cx<T> sh[hy_lds<T, PL, WMAX, OP, LP>()];
    const int64_t bid = SHORT                 ? la_pair_order(blockIdx.x, a.nrows, 2 * a.xg)
                        : LP && a.nrows == 1 ? xcd_tile_order(blockIdx.x, gridDim.x, a.xg)
                                             : blockIdx.x;
    const int tid = threadIdx.x, p = tid % WMAX, t = tid / WMAX, W = a.W;
    const int64_t nrows = a.nrows, M = a.M;
    const SlotInfo si = la_slot<ORD_XCD_ROW, false>(nrows, a.tiles_per_row, W, p < W ? p : 0, bid);
    const bool valid = p < W && si.kx < M;
    auto lds = [&](int e) -> cx<T> & { return sh[pencil_slot<LP>(e) * WMAX + p]; };
    // addresses as last_axis_block: a wave-uniform part and a 32-bit offset
    const Pack &pk = a.pk;
    const int64_t estride = pk.e_stride();
    const SlotInfo s0 = la_slot<ORD_XCD_ROW, false>(nrows, a.tiles_per_row, W, 0, bid);
    const int t0 = __builtin_amdgcn_readfirstlane(t);
    const int64_t uoff = pk.at(t0, s0.row, s0.kx);
    const uint32_t loff = (uint32_t)((pk.at(t, si.row, si.kx) - uoff) * (int64_t)sizeof(cx<T>));
    auto gp = [&](const cx<T> *base, int k) -> cx<T> * {
        return reinterpret_cast<cx<T> *>(
            reinterpret_cast<char *>(const_cast<cx<T> *>(base) + uoff + (int64_t)k * estride) + loff);
    };
    // f(i, k): this thread's i-th value at an end of radix R, element t + k
    auto each = [&](auto rc, auto &&f) {
        constexpr int R = decltype(rc)::value;
#pragma unroll
        for (int b = 0; b < PL::nb(R); ++b)
            if (PL::jok(t + b * Tp, R))
#pragma unroll
                for (int r = 0; r < R; ++r) f(b * R + r, b * Tp + r * (L / R));
    };
    constexpr std::integral_constant<int, R0> in{};
    constexpr std::integral_constant<int, Rl> mid{};
    constexpr std::integral_constant<int, Rf> end{};
    auto load = [&](const cx<T> *base, int k) { return valid ? ld_grid<NT>(gp(base, k)) : cx<T>{T(0), T(0)}; };
    const HydroArgs &h = a.h;
    cx<T> v[Rmax];
    cx<T> w[OP == HYDRO_VEL ? 1 : Rmax];  // B, then the derivative
    if constexpr (OP == HYDRO_DERIV) {
        each(mid, [&](int i, int k) { v[i] = load(a.s, k); });
    } else {
        cx<T> sp[PF ? Rmax : 1];
        if constexpr (PF) each(mid, [&](int i, int k) { sp[i] = load(a.s, k); });
        each(in, [&](int i, int k) { v[i] = load(a.a, k); });
        if constexpr (OP == HYDRO_PSI) each(in, [&](int i, int k) { w[i] = load(a.b, k); });
        fft_stages<T, PL, -1>(v, t, lds, a.tw, a.lt_shift);
        if constexpr (OP == HYDRO_PSI) fft_stages<T, PL, -1>(w, t, lds, a.tw, a.lt_shift);
        const double ky = h.fk[1] * signed_index(si.row, nrows), kx = h.fk[2] * (double)si.kx, kn = h.fk[2] * (double)M;
        auto state = [&](int i, int k) {
            if constexpr (PF)
                return sp[i];
            else
                return load(a.s, k);
        };
        auto put = [&](int i, int k, cx<T> z) {
            if constexpr (OP != HYDRO_MU)
                if (valid) st_grid<NT>(gp(a.s, k), z);
            v[i] = z;
        };
        // The folded column (X0 + i XN): the mirror element -k of every operand comes from LDS, where
        // its pencil's threads leave it before any state value is replaced.
        constexpr int NA = hy_fold_arrays<T, OP>();
        auto fold = [&](int q, int arr) { return sh + (arr * 2 + (nrows == 1 || q == 0 ? 0 : 1)) * L; };
        if (si.has_pairs) {  // uniform per workgroup
            __syncthreads();
            if (si.partner >= 0 && valid)
                each(mid, [&](int i, int k) {
                    const cx<T> S = state(i, k);
                    fold(p, 0)[t + k] = v[i];
                    if constexpr (OP == HYDRO_PSI && NA == 2)
                        fold(p, 1)[t + k] = {(T)(S.x - h.dt * w[i].x), (T)(S.y - h.dt * w[i].y)};
                    else
                        fold(p, 1)[t + k] = S;
                    if constexpr (NA == 3) fold(p, 2)[t + k] = w[i];
                });
            __syncthreads();
        }
        if (si.partner >= 0) {
            if (valid)
                each(mid, [&](int i, int k) {
                    const int e = t + k, m = neg_mod<L>(e);
                    const double kz = h.fk[0] * signed_index(e, L);
                    double p0[3][2] = {}, pn[3][2] = {};  // planes X0 and XN of each operand at k
#pragma unroll
                    for (int j = 0; j < NA; ++j) {
                        const cx<T> Z = fold(p, j)[e], Zm = fold(si.partner, j)[m];
                        p0[j][0] = 0.5 * ((double)Z.x + (double)Zm.x);
                        p0[j][1] = 0.5 * ((double)Z.y - (double)Zm.y);
                        pn[j][0] = 0.5 * ((double)Z.y + (double)Zm.y);
                        pn[j][1] = 0.5 * ((double)Zm.x - (double)Z.x);
                    }
                    const double q0 = kz * kz + ky * ky, qn = q0 + kn * kn;
                    // operand 0 is the transformed input, 1 the state (2: B)
                    constexpr int o = OP == HYDRO_MU ? 0 : 1;
                    hy_mode<OP>(h, q0, p0[o], p0[1 - o], p0[2]);
                    hy_mode<OP>(h, qn, pn[o], pn[1 - o], pn[2]);
                    put(i, k, {(T)(p0[o][0] - pn[o][1]), (T)(p0[o][1] + pn[o][0])});
                });
        } else {
            each(mid, [&](int i, int k) {
                const double kz = h.fk[0] * signed_index(t + k, L);
                const double q = kz * kz + ky * ky + kx * kx;
                const cx<T> S = state(i, k);
                const double N[2] = {(double)v[i].x, (double)v[i].y}, s[2] = {(double)S.x, (double)S.y};
                double B[2] = {0.0, 0.0};
                if constexpr (OP == HYDRO_PSI) {
                    B[0] = (double)w[i].x;
                    B[1] = (double)w[i].y;
                }
                double o[2] = {OP == HYDRO_MU ? N[0] : s[0], OP == HYDRO_MU ? N[1] : s[1]};
                hy_mode<OP>(h, q, o, OP == HYDRO_MU ? s : N, B);
                put(i, k, {(T)o[0], (T)o[1]});
            });
        }
    }
    if constexpr (OP == HYDRO_DERIV || OP == HYDRO_MU)
        each(mid, [&](int i, int k) {
            const int e = t + k;
            w[i] = mul_ik(v[i], 2 * e == L ? 0.0 : h.fk[0] * signed_index(e, L));
        });
    fft_stages<T, PR, +1>(v, t, lds, a.tw, a.lt_shift);
    if (valid) each(end, [&](int i, int k) { st_grid<NT>(gp(a.o0, k), v[i]); });
    if constexpr (OP == HYDRO_DERIV || OP == HYDRO_MU) {
        fft_stages<T, PR, +1>(w, t, lds, a.tw, a.lt_shift);
        if (valid) each(end, [&](int i, int k) { st_grid<NT>(gp(a.o1, k), w[i]); });
    }
}

// y axis, inverse: dk = inv(i k data), then data = inv(data) in place.  BOTH: one read for the two, where
// a thread's registers hold both pencils; else the pencil is read again (the first read's lines are
// mostly still in the caches).
template <typename T, class PL, int WMAX, bool NT, int G, bool LP, bool BOTH>
__global__ __launch_bounds__(WMAX *PL::Tp) void hydro_y_kernel(cx<T> *data, cx<T> *dk, int W, int64_t ncols, AxisMap am,
                                                               int64_t tiles_per_batch, const cx<T> *__restrict__ tw,
                                                               int lt_shift, int xg, double fk)
{
    constexpr int L = PL::L, Tp = PL::Tp, R0 = PL::first, Rl = PL::last, Rmax = PL::Rmax, GW = WMAX / G;
    __shared__ cx<T> sh[pencil_slot<LP>(L) * GW];
    const int64_t bid = axis_tile(am, tiles_per_batch, xg);
    const int tid = threadIdx.x, p = tid % WMAX, t = tid / WMAX;
    const int64_t batch = bid / tiles_per_batch, tile = bid - batch * tiles_per_batch;
    const int64_t col = tile * W + p;
    const bool valid = p < W && col < ncols;
    const int64_t base = am.base(batch, valid ? col : 0) + am.elem(t), es = am.estride;
    auto lds = [&](int e) -> cx<T> & { return sh[pencil_slot<LP>(e) * GW + p % GW]; };
    cx<T> v[Rmax], w[BOTH ? Rmax : 1];
    auto load = [&]() {
#pragma unroll
        for (int b = 0; b < PL::nb(R0); ++b)
            if (PL::jok(t + b * Tp, R0))
#pragma unroll
                for (int r = 0; r < R0; ++r)
                    v[b * R0 + r] = valid ? ld_grid<NT>(&data[base + (int64_t)(b * Tp + r * (L / R0)) * es]) : cx<T>{T(0), T(0)};
    };
    auto deriv = [&](cx<T> *o) {
#pragma unroll
        for (int b = 0; b < PL::nb(R0); ++b)
            if (PL::jok(t + b * Tp, R0))
#pragma unroll
                for (int r = 0; r < R0; ++r) {
                    const int e = t + b * Tp + r * (L / R0);
                    o[b * R0 + r] = mul_ik(v[b * R0 + r], 2 * e == L ? 0.0 : fk * signed_index(e, L));
                }
    };
    auto inverse = [&](cx<T> *z, cx<T> *dst) {
        fft_stages<T, PL, +1, TW_STAGE, G>(z, t, lds, tw, lt_shift, p / GW);
        if (valid) {
#pragma unroll
            for (int b = 0; b < PL::nb(Rl); ++b)
                if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                    for (int r = 0; r < Rl; ++r) st_grid<NT>(&dst[base + (int64_t)(b * Tp + r * (L / Rl)) * es], z[b * Rl + r]);
        }
    };
    load();
    if constexpr (BOTH) {
        deriv(w);
        inverse(w, dk);
    } else {
        deriv(v);
        inverse(v, dk);
        load();
    }
    inverse(v, data);
}

// One group of RI rows of an inverse x pass (x c2r; DX: of i k_x of the spectrum), times the real field
// `wt`, in v; the weights are loaded with the rows, ahead of the transform.
template <typename T, class PLI, bool PAD, bool DX>
__device__ __forceinline__ void hydro_rows(cx<T> *v, const cx<T> *spec, const T *wt, int64_t rho, int64_t nrows, int t,
                                           cx<T> *rowlds, const cx<T> *__restrict__ tw, int lt_shift, T sc, const Pack &pk,
                                           double fkx)
{
    constexpr int M = PLI::L, Tp = PLI::Tp, Rl = PLI::last, Rmax = PLI::Rmax;
    const bool valid = rho < nrows;
    int64_t ibase;
    const int64_t row = pk.x_row(valid ? rho : 0, &ibase);
    auto lds = [&](int e) -> cx<T> & { return rowlds[xidx<T, M, PAD>(e)]; };
    cx<T> w[Rmax];
    const cx<T> *wr = reinterpret_cast<const cx<T> *>(wt) + row * M;
#pragma unroll
    for (int b = 0; b < PLI::nb(Rl); ++b)
        if (PLI::jok(t + b * Tp, Rl))
#pragma unroll
            for (int r = 0; r < Rl; ++r) w[b * Rl + r] = valid ? wr[t + b * Tp + r * (M / Rl)] : cx<T>{T(0), T(0)};
    x_c2r_row<T, PLI, 1, PAD, false, false, false, DX>(v, spec + ibase, valid, t, rowlds, tw, lt_shift, pk, nullptr, fkx);
    fft_stages<T, PLI, +1>(v, t, lds, tw, lt_shift);
#pragma unroll
    for (int i = 0; i < Rmax; ++i) {
        const cx<T> x = scale(v[i], sc);
        v[i] = {w[i].x * x.x, w[i].y * x.y};
    }
}

// Leaves v as reals in the row's LDS slots.
template <typename T, class PLI>
__device__ __forceinline__ void hydro_stage(const cx<T> *v, int t, cx<T> *rowlds)
{
    constexpr int M = PLI::L, Tp = PLI::Tp, Rl = PLI::last;
    __syncthreads();
#pragma unroll
    for (int b = 0; b < PLI::nb(Rl); ++b)
        if (PLI::jok(t + b * Tp, Rl))
#pragma unroll
            for (int r = 0; r < Rl; ++r) rowlds[t + b * Tp + r * (M / Rl)] = v[b * Rl + r];
}

// x passes of one wavefront per workgroup (XFused<PLI, PLF, 64>::R rows in padded LDS rows, as the fused
// pass of the plain step); a workgroup reads its rows before it writes them.  It is XFused::threads threads:
// 64 but for rows of 750 points, whose 25 threads each leave 14 lanes of the wavefront without a row.
// out = x r2c of sum_j w[j] field_j over NC components.
template <typename T, class PLI, class PLF, int NC>
__global__ __launch_bounds__((XFused<PLI, PLF, 64>::threads)) void
hydro_adv_x_kernel(HydroFlow<T> f, int64_t nrows, const cx<T> *__restrict__ tw, int lt_shift, T sc, Pack pk)
{
    using F = XFused<PLI, PLF, 64>;
    static_assert(F::ok && PLI::L == PLF::L, "schedules must share the workgroup");
    constexpr int Tp = PLI::Tp, Rmax = PLI::Rmax, RI = F::RI, RF = F::RF;
    constexpr bool PAD = is_pow2c(PLI::L);
    constexpr int LD = XPitch<T, PLI::L, PAD>::value;
    __shared__ cx<T> sh[F::R * LD];
    const int p = threadIdx.x / Tp, t = threadIdx.x - p * Tp;
    const int64_t bid = blockIdx.x;
#pragma unroll
    for (int s = 0; s < F::R / RI; ++s) {
        const int64_t rho = (bid * (F::R / RI) + s) * RI + p;
        cx<T> *rowlds = sh + (s * RI + p) * LD;
        cx<T> acc[Rmax] = {}, v[Rmax];
#pragma unroll 1
        for (int j = 0; j < NC; ++j) {  // the x component is the last
            hydro_rows<T, PLI, PAD, true>(v, f.spec[j], f.w[j], rho, nrows, t, rowlds, tw, lt_shift, sc, pk,
                                          j + 1 < NC ? 0.0 : f.fkx);
#pragma unroll
            for (int i = 0; i < Rmax; ++i) acc[i] = acc[i] + v[i];
        }
        hydro_stage<T, PLI>(acc, t, rowlds);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < F::R / RF; ++s)
        x_r2c_block<T, PLF, RF, false, PAD, false, true>(nullptr, f.out, nrows, tw, lt_shift, bid * (F::R / RF) + s,
                                                         sh + s * RF * LD, pk);
}

// spec = x r2c of wt * (x c2r of spec; DX: of i k_x spec), in place
template <typename T, class PLI, class PLF, bool DX>
__global__ __launch_bounds__((XFused<PLI, PLF, 64>::threads)) void
hydro_force_x_kernel(cx<T> *spec, const T *wt, int64_t nrows, const cx<T> *__restrict__ tw, int lt_shift, T sc,
                     Pack pk, double fkx)
{
    using F = XFused<PLI, PLF, 64>;
    static_assert(F::ok && PLI::L == PLF::L, "schedules must share the workgroup");
    constexpr int Tp = PLI::Tp, RI = F::RI, RF = F::RF;
    constexpr bool PAD = is_pow2c(PLI::L);
    constexpr int LD = XPitch<T, PLI::L, PAD>::value;
    __shared__ cx<T> sh[F::R * LD];
    const int p = threadIdx.x / Tp, t = threadIdx.x - p * Tp;
    const int64_t bid = blockIdx.x;
#pragma unroll
    for (int s = 0; s < F::R / RI; ++s) {
        cx<T> v[PLI::Rmax];
        cx<T> *rowlds = sh + (s * RI + p) * LD;
        hydro_rows<T, PLI, PAD, DX>(v, spec, wt, (bid * (F::R / RI) + s) * RI + p, nrows, t, rowlds, tw, lt_shift, sc, pk, fkx);
        hydro_stage<T, PLI>(v, t, rowlds);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < F::R / RF; ++s)
        x_r2c_block<T, PLF, RF, false, PAD, false, true>(nullptr, spec, nrows, tw, lt_shift, bid * (F::R / RF) + s,
                                                         sh + s * RF * LD, pk);
}

// real = x c2r of in, out = x r2c of real^3
template <typename T, class PLI, class PLF>
__global__ __launch_bounds__((XFused<PLI, PLF, 64>::threads)) void
hydro_psi_x_kernel(const cx<T> *in, T *real, cx<T> *out, int64_t nrows, const cx<T> *__restrict__ tw, int lt_shift,
                   T sc, Pack pk)
{
    constexpr bool PAD = is_pow2c(PLI::L);
    __shared__ cx<T> sh[XFused<PLI, PLF, 64>::R * XPitch<T, PLI::L, PAD>::value];
    x_c2r_r2c_block<T, PLI, PLF, 64, false, PAD, false, true>(in, out, nrows, tw, lt_shift, sc, blockIdx.x, sh, pk,
                                                              (int)threadIdx.x, real);
}

// ------------------------------------------------------------------------------------------------
// Launchers.

template <typename T, int OP>
hipError_t hydro_last_op(const Geom &g, HydroLastArgs<T> a, hipStream_t s)
{
    return by_length(g.n0, [&](auto Lc) -> hipError_t {
        constexpr int L = decltype(Lc)::value;
        if constexpr (!axis_length(L)) {
            return hipErrorInvalidValue;
        } else {
            auto run = [&](auto plc, auto wc, auto lpc, auto ntc, auto shortc) -> hipError_t {
                using PL = decltype(plc);
                constexpr int WM = decltype(wc)::value;
                if (!z_steps_ok<PL>(g.zs)) return hipErrorInvalidValue;
                a.W = even_width(g.M < WM ? (int)g.M : WM);
                a.tiles_per_row = (int)cdiv(g.M, a.W);
                a.xg = line_group<T>(a.W);
                if (decltype(shortc)::value && (g.nrows == 1 || a.tiles_per_row != 1)) return hipErrorInvalidValue;
                hipLaunchKernelGGL((hydro_last_kernel<T, PL, WM, OP, decltype(ntc)::value, decltype(lpc)::value,
                                                      decltype(shortc)::value>),
                                   dim3((unsigned)(g.nrows * a.tiles_per_row)), dim3(WM * PL::Tp), 0, s, a);
                return hipGetLastError();
            };
            auto narrow = [&](auto plc) -> hipError_t {
                return run(plc, std::integral_constant<int, NarrowTile<decltype(plc)>::W>{}, std::true_type{},
                           std::false_type{}, std::false_type{});
            };
            using P3 = typename AxisPlan<L>::type;
            constexpr std::integral_constant<int, WMax<T, L>::value> wm{};
            // 2D grids never have kFillTiles tiles
            if (g.ndim == 2) return narrow(typename Last2Plan<L>::type{});
            const int W = even_width(g.M < wm.value ? (int)g.M : wm.value);
            if (g.nrows * cdiv(g.M, W) < kFillTiles) return narrow(P3{});
            // Rows of a quarter of a line at most (x = 4, FP32 also 8) would leave most of the tile's lanes idle, and
            // from 256 points up that shows: tiles of a row's half and its mirror's, mixed lengths over more
            // threads as in 2D.  Two steps, in ms, of separate passes (whose tiles cross rows), full tiles, these:
            // 1024 x 1024 x 8 FP32 2.77, 3.95, 2.69, 1400 x 1400 x 8 7.20, 9.27, 6.47, 700 x 2048 x 4 3.12, 5.55,
            // 3.14, FP64 2.94, 4.13, 2.60; 1024 x 2048 x 4 FP32 4.11, 7.03, 4.61 and 2048 x 2048 x 4 8.16, 9.17,
            // 9.21, where the folded pencils' LDS leaves one to three workgroups per CU.
            if constexpr (L >= 256) {
                using PS = std::conditional_t<is_pow2c(L), P3, typename Last2Plan<L>::type>;
                auto rows_of = [&](auto wc) {
                    return run(PS{}, wc, std::true_type{}, std::false_type{}, std::true_type{});
                };
                if (g.M == 2) return rows_of(std::integral_constant<int, 2>{});
                if constexpr (sizeof(T) == 4)
                    if (g.M == 4) return rows_of(std::integral_constant<int, 4>{});
            }
            return with_nt<line_group<T>(even_width(wm.value)) == 1>(g.nt && line_group<T>(W) == 1,
                           [&](auto ntc) -> hipError_t { return run(P3{}, wm, std::false_type{}, ntc, std::false_type{}); });
        }
    });
}

template <typename T>
HydroLastArgs<T> hydro_last_args(const Geom &g, const cx<T> *a, const cx<T> *b, cx<T> *s, cx<T> *o0, cx<T> *o1,
                                 const HydroArgs &h, const cx<T> *tw)
{
    HydroLastArgs<T> r{};
    r.a = a;
    r.b = b;
    r.s = s;
    r.o0 = o0;
    r.o1 = o1;
    r.nrows = g.nrows;
    r.M = (int)g.M;
    r.tw = tw + g.tw_last;
    r.lt_shift = g.lt_shift;
    r.h = h;
    r.pk = pack_of(g);
    return r;
}

template <typename T>
hipError_t launch_hydro_y(const Geom &g, cx<T> *data, cx<T> *dk, double fk, const cx<T> *tw, hipStream_t s)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    return by_length(g.n1, [&](auto Lc) -> hipError_t {
        constexpr int L = decltype(Lc)::value;
        if constexpr (!axis_length(L)) {
            return hipErrorInvalidValue;
        } else {
            using TO = TileOf<T, typename ListAt<0, typename AxisCands<L>::type>::type>;
            using TL = typename TO::tile;
            using PL = SpreadIf<typename TO::plan, TL::E>;
            using PN = typename TO::plan;
            constexpr int WM = TL::W, WN = NarrowTile<PN>::W;
            const int W = (int)(g.M < WM ? g.M : WM);
            const int64_t tiles = cdiv(g.M, W);
            const AxisMap am = y_map(g);
            if constexpr (WN < WM) {
                if (tiles * g.n0 < kFillTiles) {  // two transforms, as launch_y_c2c otherwise
                    const int w = (int)(g.M < WN ? g.M : WN);
                    const int64_t nt = cdiv(g.M, w);
                    hipLaunchKernelGGL((hydro_y_kernel<T, PN, WN, false, 1, true, true>), dim3((unsigned)(nt * g.n0)),
                                       dim3(WN * PN::Tp), 0, s, data, dk, w, g.M, am, nt, tw + g.tw_y, g.lt_shift,
                                       line_group<T>(w), fk);
                    return hipGetLastError();
                }
            }
            const int xg = (line_group<T>(W) == 1 && (TL::G == 1 || !is_pow2c(L))) ? 0 : line_group<T>(W);
            constexpr bool BOTH = TL::G == 1 && PL::Rmax <= 20;
            return with_nt<BOTH && line_group<T>(WM) == 1>(g.nt && xg <= 1, [&](auto ntc) -> hipError_t {
                hipLaunchKernelGGL((hydro_y_kernel<T, PL, WM, decltype(ntc)::value, TL::G, false, BOTH>),
                                   dim3((unsigned)(tiles * g.n0)), dim3(WM * PL::Tp), 0, s, data, dk, W, g.M, am, tiles,
                                   tw + g.tw_y, g.lt_shift, xg, fk);
                return hipGetLastError();
            });
        }
    });
}

// Calls f(PLI{}, PLF{}) with the x schedules of both directions: TWO those of the 2D lists.
template <bool TWO, class F>
hipError_t with_x_plans(const Geom &g, F &&f)
{
    return by_length(g.M, [&](auto Mc) -> hipError_t {
        constexpr int M = decltype(Mc)::value;
        if constexpr (M > 1024) {
            return hipErrorInvalidValue;
        } else {
            if (TWO || g.ndim == 2) return f(typename X2InvPlan<M>::type{}, typename X2FwdPlan<M>::type{});
            return f(typename XInvPlan<M>::type{}, typename XFwdPlan<M>::type{});
        }
    });
}

template <typename T>
hipError_t launch_hydro_x(const Geom &g, const HydroFlow<T> &fl, const cx<T> *tw, hipStream_t s)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    const T sc = (T)(1.0 / ((double)g.M * (double)g.n0 * (double)g.nrows));
    const Pack pk = pack_of(g);
    const cx<T> *twx = tw + g.tw_x;
    if (fl.out)  // three components' registers: the schedules of 8 elements per thread in both directions
        return with_x_plans<true>(g, [&](auto pic, auto pfc) -> hipError_t {
            using PLI = decltype(pic);
            using PLF = decltype(pfc);
            const dim3 grid((unsigned)cdiv(g.xrows, XFused<PLI, PLF, 64>::R)), block(XFused<PLI, PLF, 64>::threads);
            if (g.ndim == 3)
                hipLaunchKernelGGL((hydro_adv_x_kernel<T, PLI, PLF, 3>), grid, block, 0, s, fl, g.xrows, twx, g.lt_shift, sc, pk);
            else
                hipLaunchKernelGGL((hydro_adv_x_kernel<T, PLI, PLF, 2>), grid, block, 0, s, fl, g.xrows, twx, g.lt_shift, sc, pk);
            return hipGetLastError();
        });
    // one launch per component: all in one kernel took 104 registers a thread instead of 60, half the
    // wavefronts, and 2.15 ms at 512^3 FP32
    return with_x_plans<false>(g, [&](auto pic, auto pfc) -> hipError_t {
        using PLI = decltype(pic);
        using PLF = decltype(pfc);
        const dim3 grid((unsigned)cdiv(g.xrows, XFused<PLI, PLF, 64>::R)), block(XFused<PLI, PLF, 64>::threads);
        for (int j = 0; j < g.ndim; ++j) {
            if (j + 1 < g.ndim)
                hipLaunchKernelGGL((hydro_force_x_kernel<T, PLI, PLF, false>), grid, block, 0, s, fl.spec[j], fl.w[0], g.xrows,
                                   twx, g.lt_shift, sc, pk, 0.0);
            else
                hipLaunchKernelGGL((hydro_force_x_kernel<T, PLI, PLF, true>), grid, block, 0, s, fl.spec[j], fl.w[0], g.xrows,
                                   twx, g.lt_shift, sc, pk, fl.fkx);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    });
}

template <typename T>
hipError_t launch_hydro_psi_x(const Geom &g, const cx<T> *in, T *real, cx<T> *out, const cx<T> *tw, hipStream_t s)
{
    if (!layout_ok(g)) return hipErrorInvalidValue;
    return with_x_plans<false>(g, [&](auto pic, auto pfc) -> hipError_t {
        using PLI = decltype(pic);
        using PLF = decltype(pfc);
        const T sc = (T)(1.0 / ((double)g.M * (double)g.n0 * (double)g.nrows));
        using F = XFused<PLI, PLF, 64>;
        hipLaunchKernelGGL((hydro_psi_x_kernel<T, PLI, PLF>), dim3((unsigned)cdiv(g.xrows, F::R)), dim3(F::threads), 0, s, in,
                           real, out, g.xrows, tw + g.tw_x, g.lt_shift, sc, pack_of(g));
        return hipGetLastError();
    });
}

}  // namespace pfc
