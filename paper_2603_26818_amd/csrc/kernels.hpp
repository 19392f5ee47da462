// kernels.hpp -- HIP kernels of the PFC hot path (gfx950).
//
// Layouts (C-order, x fastest; M = n_x / 2):
//   real field      [rows][2M]                      rows = n0 n1 (3D) or n0 (2D)
//   packed spectrum [n0][nrows][M] complex           nrows = n1 (3D) or 1 (2D)
//     column kx in 1..M-1 holds X(kx); column 0 holds X(0) + i X(M): the planes kx = 0 and
//     kx = n_x/2 are spectra of real data and share one complex plane.  After the transforms along
//     the other axes, column 0 holds Z = X0_hat + i XN_hat, and the two Hermitian planes are
//         X0_hat(k) = (Z(k) + conj Z(-k)) / 2,   XN_hat(k) = -i (Z(k) - conj Z(-k)) / 2.
//   natural half    [n0][nrows][M+1] complex
//
// Pass schedule of one step (arxiv 2603.26818, Listing 1: cube, forward transform, update of the
// spectrum, inverse transform), 3D:
//   x_r2c (cube prologue) -> y forward -> last-axis (z forward, update, z inverse) -> y inverse
//   -> x_c2r (1/N epilogue);   2D: x_r2c -> last-axis along y -> x_c2r.
#pragma once

#include "fft_core.hpp"

namespace pfc {

// ------------------------------------------------------------------------------------------------
// L(q) and the implicit multiplier, in the kernel's precision (ModelParams in types.hpp).
template <typename T>
__device__ __forceinline__ T corr_op(const ModelParams<T> &m, T q)
{
    T a = (T(1) - q) * (T(1) - q);
    if (m.model == 0) return a;
    T b = m.q1sq - q;
    return a * (b * b + m.R1);
}

// A(q) = 1 / (1 + dt q (r + L(q))); exactly 1 at q = 0.  FP32 takes the hardware reciprocal
// (within 1 ulp, exact for 1); FP64 divides.
template <typename T>
__device__ __forceinline__ T amult(const ModelParams<T> &m, T q)
{
    const T d = T(1) + m.dt * q * (m.r + corr_op(m, q));
    if constexpr (sizeof(T) == 4)
        return __builtin_amdgcn_rcpf(d);
    else
        return T(1) / d;
}

// Loads and stores of the streamed grids.  NT marks them non-temporal: on grids far larger than
// the caches, nothing a pass touches is read again before it is evicted.
template <bool NT, typename T>
__device__ __forceinline__ cx<T> ld_grid(const cx<T> *p)
{
    if constexpr (NT) {
        typedef T v2 __attribute__((ext_vector_type(2)));
        const v2 v = __builtin_nontemporal_load(reinterpret_cast<const v2 *>(p));
        return {v.x, v.y};
    } else {
        return *p;
    }
}
template <bool NT, typename T>
__device__ __forceinline__ void st_grid(cx<T> *p, cx<T> a)
{
    if constexpr (NT) {
        typedef T v2 __attribute__((ext_vector_type(2)));
        v2 v;
        v.x = a.x;
        v.y = a.y;
        __builtin_nontemporal_store(v, reinterpret_cast<v2 *>(p));
    } else {
        *p = a;
    }
}

// i k z in FP64, rounded once: a spectral derivative
template <typename T>
__device__ __forceinline__ cx<T> mul_ik(cx<T> z, double k)
{
    return {(T)(-k * (double)z.y), (T)(k * (double)z.x)};
}

__device__ __forceinline__ int signed_index(int64_t i, int64_t n) { return (int)(i <= n / 2 ? i : i - n); }

// (-e) mod L for 0 <= e < L
template <int L>
__device__ __forceinline__ int neg_mod(int e)
{
    if constexpr (is_pow2c(L))
        return (L - e) & (L - 1);
    else
        return e == 0 ? 0 : L - e;
}

// x-pass split twiddle W_{2M}^k, 0 <= k < M: from the W_Lt table, or from the length's own table
// (lengths that are not powers of two; layout in fft_core.hpp)
template <typename T, int M>
__device__ __forceinline__ cx<T> split_twiddle(const cx<T> *__restrict__ tw, int lt_shift, int k)
{
    if constexpr (is_pow2c(M))
        return tw[k << (lt_shift - ilog2c(2 * M))];
    else
        return tw[MixTable<M>::split + k];
}

// ------------------------------------------------------------------------------------------------
// Block-wide FP64 sum; the result is valid in thread 0.  red: >= blockDim.x/64 doubles of LDS.
__device__ __forceinline__ double block_sum(double v, double *red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)(blockDim.x + 63) / 64; ++i) s += red[i];
    return s;
}

// ------------------------------------------------------------------------------------------------
// x axis, forward: one row of 2M reals -> M packed complex values.
// z[m] = x[2m] + i x[2m+1] (cubed first when CUBE), Z = FFT_M(z), then for k = 1..M-1
//   X(k) = E + W_{2M}^k O,  E = (Z(k) + conj Z(M-k)) / 2,  O = -i (Z(k) - conj Z(M-k)) / 2,
// and slot 0 = (Re Z0 + Im Z0) + i (Re Z0 - Im Z0) = X(0) + i X(M).
// rows per workgroup of the x pass: about 256 threads
template <class PL>
struct XRows {
    static constexpr int value = (256 / PL::Tp) > 64 ? 64 : ((256 / PL::Tp) < 1 ? 1 : 256 / PL::Tp);
};

// Padded LDS rows of the x pass (PAD, power-of-two rows of M complex values): 16 spare bytes after
// every 256 bytes of a row, i.e. after every S = 256 / sizeof(cx<T>) elements (M, if shorter).  With
// 64 banks of 4 bytes, a Stockham stage write puts neighbouring threads R elements apart; unpadded,
// the threads of a power-of-two row then meet on a few bank positions of each 256-byte sweep (up to
// 16 ways for the first stage of a 512-point r2c).  The 16-byte step keeps 16-byte alignment and
// fixed offsets between one thread's elements, so merged and paired LDS accesses stay possible.
template <typename T, int M>
struct XPad {
    static constexpr int S0 = 256 / (int)sizeof(cx<T>);
    static constexpr int S = S0 < M ? S0 : M;
    static constexpr int k = 16 / (int)sizeof(cx<T>);
    static constexpr int shift = ilog2c(S);
};
template <typename T, int M, bool PAD>
struct XPitch {
    static_assert(!PAD || is_pow2c(M), "padded rows are powers of two");
    static constexpr int value = PAD ? M + XPad<T, M>::k * (M / XPad<T, M>::S) : M;
};
template <typename T, int M, bool PAD>
__device__ __forceinline__ int xidx(int e)
{
    if constexpr (PAD)
        return e + XPad<T, M>::k * (e >> XPad<T, M>::shift);
    else
        return e;
}

// Identity layout of a packed spectrum with rows of M values (2D plans, the batched form).
__host__ __device__ inline Pack row_pack(int64_t M) { return Pack{1, M, 0, 0}; }

// Twiddles of an x pass loaded ahead (see StageTw): the stages', and the split twiddles W_{2M}^k of the
// elements a thread holds at the real end (last radix of the r2c, FWD; first of the c2r).
template <typename T, class PL>
struct XTw {
    StageTw<T, PL> st;
    cx<T> split[PL::Rmax];
};
template <typename T, class PL, bool FWD>
__device__ __forceinline__ void load_xtw(XTw<T, PL> &o, int t, const cx<T> *__restrict__ tw, int lt_shift)
{
    load_stage_tw<T, PL, FWD ? TW_LT : TW_STAGE>(o.st, t, tw, lt_shift);
    constexpr int R = FWD ? PL::last : PL::first;
#pragma unroll
    for (int b = 0; b < PL::nb(R); ++b)
        if (PL::jok(t + b * PL::Tp, R))
#pragma unroll
            for (int r = 0; r < R; ++r)
                o.split[b * R + r] = split_twiddle<T, PL::L>(tw, lt_shift, t + b * PL::Tp + r * (PL::L / R));
}

// One block of ROWS rows (block index `bid`); `sh` holds ROWS * XPitch<T, M, PAD> LDS slots.
// Uses threads 0 .. ROWS*Tp-1, which must be all threads of the workgroup.  FROM_LDS: the rows'
// reals are not read from `in` but from `sh` (row p at sh[p LD], LD the row pitch, as packed
// pairs, contiguous), where the caller
// has left them.  Output row rr (= e nrows + row) goes to the layout `pk`.
// PRE: the twiddles come from `pre` (load_xtw).
template <typename T, class PL, int ROWS, bool CUBE, bool PAD = false, bool NT = false, bool FROM_LDS = false,
          bool PRE = false>
__device__ __forceinline__ void x_r2c_block(const T *__restrict__ in, cx<T> *__restrict__ out, int64_t nrows,
                                            const cx<T> *__restrict__ tw, int lt_shift, int64_t bid, cx<T> *sh,
                                            const Pack &pk, const int tid = (int)threadIdx.x,
                                            const XTw<T, PL> *pre = nullptr)
{
    constexpr int M = PL::L, Tp = PL::Tp, R0 = PL::first, Rl = PL::last, Rmax = PL::Rmax;
    constexpr int LD = XPitch<T, M, PAD>::value;  // row pitch in LDS
    const int p = tid / Tp, t = tid - p * Tp;
    const int64_t rho = bid * ROWS + p;  // position in the pass's row order (Pack::x_row)
    const bool valid = rho < nrows;
    int64_t obase;
    const int64_t row = pk.x_row(valid ? rho : 0, &obase);
    const cx<T> *src = FROM_LDS ? sh + p * LD : reinterpret_cast<const cx<T> *>(in) + row * M;
    cx<T> v[Rmax];
#pragma unroll
    for (int b = 0; b < PL::nb(R0); ++b)
        if (PL::jok(t + b * Tp, R0))
#pragma unroll
        for (int r = 0; r < R0; ++r) {
            cx<T> z;
            if constexpr (FROM_LDS)
                z = src[t + b * Tp + r * (M / R0)];
            else
                z = valid ? ld_grid<NT>(&src[t + b * Tp + r * (M / R0)]) : cx<T>{T(0), T(0)};
            if constexpr (CUBE) z = {z.x * z.x * z.x, z.y * z.y * z.y};
            v[b * R0 + r] = z;
        }
    auto lds = [&](int e) -> cx<T> & { return sh[p * LD + xidx<T, M, PAD>(e)]; };
    // measured faster here than TW_STAGE
    fft_stages<T, PL, -1, TW_LT, 1, PRE>(v, t, lds, tw, lt_shift, 0, PRE ? &pre->st : nullptr);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < PL::nb(Rl); ++b)
        if (PL::jok(t + b * Tp, Rl))
#pragma unroll
        for (int r = 0; r < Rl; ++r) lds(t + b * Tp + r * (M / Rl)) = v[b * Rl + r];
    __syncthreads();
    cx<T> *dst = out + obase;
    const T h = T(0.5);
#pragma unroll
    for (int b = 0; b < PL::nb(Rl); ++b)
        if (PL::jok(t + b * Tp, Rl))
#pragma unroll
        for (int r = 0; r < Rl; ++r) {
            const int k = t + b * Tp + r * (M / Rl);
            const cx<T> Zk = v[b * Rl + r];
            cx<T> X;
            if (k == 0) {
                X = {Zk.x + Zk.y, Zk.x - Zk.y};
            } else {
                const cx<T> Zp = lds(M - k);
                const cx<T> E = {(Zk.x + Zp.x) * h, (Zk.y - Zp.y) * h};
                const cx<T> O = {(Zk.y + Zp.y) * h, (Zp.x - Zk.x) * h};
                X = E + cmul(PRE ? pre->split[b * Rl + r] : split_twiddle<T, M>(tw, lt_shift, k), O);
            }
            if (valid) st_grid<NT>(&dst[pk.col(k)], X);
        }
}

template <typename T, class PL, int ROWS, bool CUBE, bool PAD = false, bool NT = false, bool LAT = false>
__global__ __launch_bounds__(ROWS *PL::Tp) void x_r2c_kernel(const T *__restrict__ in, cx<T> *__restrict__ out,
                                                              int64_t nrows, const cx<T> *__restrict__ tw,
                                                              int lt_shift, Pack pk)
{
    __shared__ cx<T> sh[ROWS * XPitch<T, PL::L, PAD>::value];
    constexpr bool PRE = LAT && preload_tw<T, PL>();
    XTw<T, PL> pre;
    if constexpr (PRE) load_xtw<T, PL, true>(pre, (int)threadIdx.x % PL::Tp, tw, lt_shift);
    x_r2c_block<T, PL, ROWS, CUBE, PAD, NT, false, PRE>(in, out, nrows, tw, lt_shift, blockIdx.x, sh, pk,
                                                        (int)threadIdx.x, &pre);
}

// ------------------------------------------------------------------------------------------------
// x axis, inverse: M packed complex -> 2M reals (times `scale`).  For k = 1..M-1
//   E = (X(k) + conj X(M-k)) / 2,  O = conj(W_{2M}^k) (X(k) - conj X(M-k)) / 2,  Z(k) = E + i O,
// Z(0) = ((X0 + XM) + i (X0 - XM)) / 2 from the packed slot; z = IFFT_M(Z) (unnormalised);
// x[2m] = Re z[m] * scale, x[2m+1] = Im z[m] * scale.
//
// EPI_PLAIN stores x.  EPI_ADJOINT transforms two spectra (mu from `in`, in the layout `pk`; nu
// from `in2`, always in the plain layout of rows of M, so that nu's row r covers the same bytes as
// the real row r) and stores
//   out = mu - c3 * psi_n^2 * nu   (TO_LDS: to the rows' LDS slots, as EPI_PLAIN), adding the thread's FP64
// share of the sum of nu * psi_np1 to *acc, whose workgroup sum goes to partial[bid] (adj_partial).
// `in2` and `out` may be the same buffer: each block reads its rows completely before writing them.
enum { EPI_PLAIN = 0, EPI_ADJOINT = 1 };

template <typename T>
struct AdjEpi {
    const cx<T> *in2;
    const T *psi_n;
    const T *psi_np1;
    T c3;
    double *partial;
    int add;  // partial[bid] += the sum, instead of =
};

// The workgroup's sum of acc to its own slot of the partials.
template <typename T>
__device__ __forceinline__ void adj_partial(const AdjEpi<T> &ea, double acc, int64_t bid)
{
    __shared__ double red[16];
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) ea.partial[bid] = ea.add ? ea.partial[bid] + s : s;
}

// Pre-combination of one row for the c2r: own elements X(k) from `src` (column k at src[pk.col(k)]);
// the mirror X(M-k) either through LDS (PG = false) or straight from `src` (PG = true: a second,
// reversed but coalesced load of the same cache lines, without the LDS round trip and its barrier).
// DX: X(k) is replaced by i (k fkx) X(k), the spectral x derivative (0 for the planes k = 0 and k = M
// of slot 0), computed in FP64 and rounded once, unless fkx is 0.
template <typename T, class PL, int ROWS, bool PAD, bool PG = false, bool NT = false, bool PRE = false, bool DX = false>
__device__ __forceinline__ void x_c2r_row(cx<T> *v, const cx<T> *src, bool valid, int t, cx<T> *rowlds,
                                          const cx<T> *__restrict__ tw, int lt_shift, const Pack &pk,
                                          const XTw<T, PL> *pre = nullptr, double fkx = 0.0)
{
    constexpr int M = PL::L, Tp = PL::Tp, R0 = PL::first, Rmax = PL::Rmax;
    cx<T> mir[PG ? Rmax : 1];
    if constexpr (PG) {
#pragma unroll
        for (int b = 0; b < PL::nb(R0); ++b)
            if (PL::jok(t + b * Tp, R0))
#pragma unroll
            for (int r = 0; r < R0; ++r) {
                const int k = t + b * Tp + r * (M / R0);
                v[b * R0 + r] = valid ? ld_grid<NT>(&src[pk.col(k)]) : cx<T>{T(0), T(0)};
                mir[b * R0 + r] = valid ? ld_grid<NT>(&src[pk.col(neg_mod<M>(k))]) : cx<T>{T(0), T(0)};
            }
    } else {
        __syncthreads();
#pragma unroll
        for (int b = 0; b < PL::nb(R0); ++b)
            if (PL::jok(t + b * Tp, R0))
#pragma unroll
            for (int r = 0; r < R0; ++r) {
                const int k = t + b * Tp + r * (M / R0);
                v[b * R0 + r] = valid ? ld_grid<NT>(&src[pk.col(k)]) : cx<T>{T(0), T(0)};
                if constexpr (DX)
                    if (fkx != 0.0) v[b * R0 + r] = mul_ik(v[b * R0 + r], fkx * (double)k);
                rowlds[xidx<T, M, PAD>(k)] = v[b * R0 + r];
            }
        __syncthreads();
    }
    const T h = T(0.5);
#pragma unroll
    for (int b = 0; b < PL::nb(R0); ++b)
        if (PL::jok(t + b * Tp, R0))
#pragma unroll
        for (int r = 0; r < R0; ++r) {
            const int k = t + b * Tp + r * (M / R0);
            const cx<T> a = v[b * R0 + r];
            if (k == 0) {
                v[b * R0 + r] = {(a.x + a.y) * h, (a.x - a.y) * h};
            } else {
                cx<T> c;  // X(M-k); conj taken below
                if constexpr (PG)
                    c = mir[b * R0 + r];
                else
                    c = rowlds[xidx<T, M, PAD>(M - k)];
                const cx<T> E = {(a.x + c.x) * h, (a.y - c.y) * h};
                const cx<T> D = {(a.x - c.x) * h, (a.y + c.y) * h};
                const cx<T> O = cmul(conj(PRE ? pre->split[b * R0 + r] : split_twiddle<T, M>(tw, lt_shift, k)), D);
                v[b * R0 + r] = {E.x - O.y, E.y + O.x};
            }
        }
}

// TO_LDS (EPI_PLAIN): the scaled reals of row p are left in sh[p LD] (LD the row pitch, as packed
// pairs, contiguous) instead of being stored to `out` (STORE: as well as).
template <typename T, class PL, int ROWS, int EPI, bool PAD = false, bool PG = false, bool NT = false,
          bool TO_LDS = false, bool PRE = false, bool STORE = false>
__device__ __forceinline__ void x_c2r_block(const cx<T> *in, T *out, int64_t nrows, const cx<T> *__restrict__ tw,
                                            int lt_shift, T sc, const AdjEpi<T> &ea, int64_t bid, cx<T> *sh,
                                            const Pack &pk, const int tid = (int)threadIdx.x,
                                            const XTw<T, PL> *pre = nullptr, double *acc = nullptr)
{
    constexpr int M = PL::L, Tp = PL::Tp, Rl = PL::last, Rmax = PL::Rmax;
    constexpr int LD = XPitch<T, M, PAD>::value;
    const int p = tid / Tp, t = tid - p * Tp;
    const int64_t rho = bid * ROWS + p;  // position in the pass's row order (Pack::x_row)
    const bool valid = rho < nrows;
    int64_t ibase;
    const int64_t r0 = pk.x_row(valid ? rho : 0, &ibase);  // real-field row
    auto lds = [&](int e) -> cx<T> & { return sh[p * LD + xidx<T, M, PAD>(e)]; };
    cx<T> v[Rmax];
    x_c2r_row<T, PL, ROWS, PAD, PG, NT, PRE>(v, in + ibase, valid, t, &sh[p * LD], tw, lt_shift, pk, pre);
    fft_stages<T, PL, +1, TW_STAGE, 1, PRE>(v, t, lds, tw, lt_shift, 0, PRE ? &pre->st : nullptr);
    cx<T> *dst = reinterpret_cast<cx<T> *>(out) + r0 * M;
    if constexpr (EPI == EPI_PLAIN && TO_LDS) {
        __syncthreads();  // every thread of the row is past its last exchange read
#pragma unroll
        for (int b = 0; b < PL::nb(Rl); ++b)
            if (PL::jok(t + b * Tp, Rl))
#pragma unroll
            for (int r = 0; r < Rl; ++r) {
                const cx<T> x = scale(v[b * Rl + r], sc);
                sh[p * LD + t + b * Tp + r * (M / Rl)] = x;
                if constexpr (STORE)
                    if (valid) st_grid<NT>(&dst[t + b * Tp + r * (M / Rl)], x);
            }
    } else if constexpr (EPI == EPI_PLAIN) {
        if (valid) {
#pragma unroll
            for (int b = 0; b < PL::nb(Rl); ++b)
                if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                for (int r = 0; r < Rl; ++r)
                    st_grid<NT>(&dst[t + b * Tp + r * (M / Rl)], scale(v[b * Rl + r], sc));
        }
    } else {
        cx<T> w[Rmax];
        x_c2r_row<T, PL, ROWS, PAD, PG, false, PRE>(w, ea.in2 + r0 * M, valid, t, &sh[p * LD], tw, lt_shift,
                                                    row_pack(M), pre);
        fft_stages<T, PL, +1, TW_STAGE, 1, PRE>(w, t, lds, tw, lt_shift, 0, PRE ? &pre->st : nullptr);
        const cx<T> *pn = reinterpret_cast<const cx<T> *>(ea.psi_n) + r0 * M;
        const cx<T> *pn1 = reinterpret_cast<const cx<T> *>(ea.psi_np1) + r0 * M;
        if constexpr (TO_LDS) __syncthreads();  // every thread of the row is past its last exchange read
        if (valid) {
#pragma unroll
            for (int b = 0; b < PL::nb(Rl); ++b)
                if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                for (int r = 0; r < Rl; ++r) {
                    const int m = t + b * Tp + r * (M / Rl);
                    const cx<T> mu = scale(v[b * Rl + r], sc), nu = scale(w[b * Rl + r], sc);
                    const cx<T> a = pn[m], c = pn1[m];
                    const cx<T> o = {mu.x - ea.c3 * a.x * a.x * nu.x, mu.y - ea.c3 * a.y * a.y * nu.y};
                    if constexpr (TO_LDS)
                        sh[p * LD + m] = o;
                    else
                        dst[m] = o;
                    *acc += (double)nu.x * (double)c.x + (double)nu.y * (double)c.y;
                }
        }
    }
}

template <typename T, class PL, int ROWS, int EPI, bool PAD = false, bool PG = false, bool NT = false, bool LAT = false>
__global__ __launch_bounds__(ROWS *PL::Tp) void x_c2r_kernel(const cx<T> *in, T *out, int64_t nrows,
                                                              const cx<T> *__restrict__ tw, int lt_shift, T sc,
                                                              AdjEpi<T> ea, Pack pk)
{
    __shared__ cx<T> sh[ROWS * XPitch<T, PL::L, PAD>::value];
    constexpr bool PRE = LAT && preload_tw<T, PL>();
    XTw<T, PL> pre;
    if constexpr (PRE) load_xtw<T, PL, false>(pre, (int)threadIdx.x % PL::Tp, tw, lt_shift);
    double acc = 0.0;
    x_c2r_block<T, PL, ROWS, EPI, PAD, PG, NT, false, PRE>(in, out, nrows, tw, lt_shift, sc, ea, blockIdx.x, sh, pk,
                                                           (int)threadIdx.x, &pre, &acc);
    if constexpr (EPI == EPI_ADJOINT) adj_partial(ea, acc, blockIdx.x);
}

// ------------------------------------------------------------------------------------------------
// x pass between two steps (batched runs, and the single-plan step within one call): the inverse x
// transform of one step (x c2r) and the forward x transform with the cube of the next (x r2c), over
// the same rows, with the field between them kept in LDS: a workgroup takes R rows, runs the c2r
// schedule PLI on them in groups of RI rows (each group leaving its reals in its rows' LDS slots),
// then the r2c schedule PLF in groups of RF rows reading those slots.  The field of the intermediate
// step is never stored.  Arithmetic identical to x_c2r_kernel followed by x_r2c_kernel with the
// cube.  The single-plan step runs it with one wavefront per workgroup (at 512^3: 4 rows in padded
// LDS rows, 8.5 KB, many workgroups per CU), which keeps the row FFTs, that bound it at half the
// memory traffic, overlapped; 256-thread workgroups measured no faster than the two separate passes.
template <class PLI, class PLF, int NTH = 256>
struct XFused {
    static constexpr int RI = NTH / PLI::Tp < 1 ? 1 : NTH / PLI::Tp;
    static constexpr int RF = NTH / PLF::Tp < 1 ? 1 : NTH / PLF::Tp;
    static constexpr int R = RI > RF ? RI : RF;
    static constexpr int threads = RI * PLI::Tp;
    // both schedules fill the same workgroup, and a group of either kind tiles the R rows
    static constexpr bool ok = RI * PLI::Tp == RF * PLF::Tp && R % RI == 0 && R % RF == 0;
};
// One block of R rows (block index `bid`) of packed spectra in the layout `pk`; `sh` holds
// R XPitch<T, M, PAD> LDS slots; exactly XFused<PLI, PLF, NTH>::threads threads (fewer than NTH where the
// threads per row do not divide it: a thread past them would take a row of the next workgroup).  In place
// (in == out) is safe: the block reads all its rows before it writes.  STORE: the field in between is also
// stored, to `real`.
template <typename T, class PLI, class PLF, int NTH, bool NT = false, bool PAD = false, bool LAT = false, bool STORE = false>
__device__ __forceinline__ void x_c2r_r2c_block(const cx<T> *in, cx<T> *out, int64_t nrows,
                                                const cx<T> *__restrict__ tw, int lt_shift, T sc, int64_t bid,
                                                cx<T> *sh, const Pack &pk, const int tid = (int)threadIdx.x,
                                                T *real = nullptr)
{
    using F = XFused<PLI, PLF, NTH>;
    static_assert(F::ok && PLI::L == PLF::L, "schedules must share the workgroup");
    constexpr int LD = XPitch<T, PLI::L, PAD>::value;
    const AdjEpi<T> ea{};
    constexpr bool PRE = LAT && preload_tw<T, PLI>() && preload_tw<T, PLF>();
    XTw<T, PLI> prei;
    XTw<T, PLF> pref;
    if constexpr (PRE) {
        load_xtw<T, PLI, false>(prei, tid % PLI::Tp, tw, lt_shift);
        load_xtw<T, PLF, true>(pref, tid % PLF::Tp, tw, lt_shift);
    }
#pragma unroll
    for (int s = 0; s < F::R / F::RI; ++s)
        x_c2r_block<T, PLI, F::RI, EPI_PLAIN, PAD, false, NT, true, PRE, STORE>(in, real, nrows, tw, lt_shift, sc, ea,
                                                                         bid * (F::R / F::RI) + s, sh + s * F::RI * LD,
                                                                         pk, tid, &prei);
    __syncthreads();  // all staged rows written
#pragma unroll
    for (int s = 0; s < F::R / F::RF; ++s)
        x_r2c_block<T, PLF, F::RF, true, PAD, NT, true, PRE>(nullptr, out, nrows, tw, lt_shift, bid * (F::R / F::RF) + s,
                                                             sh + s * F::RF * LD, pk, tid, &pref);
}

// The fused x pass of the single-plan step between two steps: one workgroup of XFused::threads threads
// (one wavefront in the step) takes XFused<PLI, PLF, NTH>::R rows of the packed spectrum, in place.
// STORE: the field in between is also stored, to `real`.
template <typename T, class PLI, class PLF, int NTH, bool NT, bool PAD, bool LAT = false, bool STORE = false>
__global__ __launch_bounds__((XFused<PLI, PLF, NTH>::threads)) void
x_c2r_r2c_kernel(cx<T> *data, T *real, int64_t nrows, const cx<T> *__restrict__ tw, int lt_shift, T sc, Pack pk)
{
    __shared__ cx<T> sh[XFused<PLI, PLF, NTH>::R * XPitch<T, PLI::L, PAD>::value];
    x_c2r_r2c_block<T, PLI, PLF, NTH, NT, PAD, LAT, STORE>(data, data, nrows, tw, lt_shift, sc, blockIdx.x, sh, pk,
                                                           (int)threadIdx.x, real);
}

// The x pass between two adjoint steps: lambda_n of one (EPI_ADJOINT) and the x r2c of lambda_n that the
// next one starts with, one wavefront per workgroup as above; lambda_n itself is not stored.  mu and the
// output spectrum are `data`.
template <typename T, class PLI, class PLF, bool PAD, bool LAT>
__global__ __launch_bounds__((XFused<PLI, PLF, 64>::threads)) void
x_adj_r2c_kernel(cx<T> *data, int64_t nrows, const cx<T> *__restrict__ tw, int lt_shift, T sc, AdjEpi<T> ea, Pack pk)
{
    using F = XFused<PLI, PLF, 64>;
    constexpr int LD = XPitch<T, PLI::L, PAD>::value;
    constexpr bool PRE = LAT && preload_tw<T, PLI>() && preload_tw<T, PLF>();
    __shared__ cx<T> sh[F::R * LD];
    XTw<T, PLI> prei;
    XTw<T, PLF> pref;
    if constexpr (PRE) {
        load_xtw<T, PLI, false>(prei, (int)threadIdx.x % PLI::Tp, tw, lt_shift);
        load_xtw<T, PLF, true>(pref, (int)threadIdx.x % PLF::Tp, tw, lt_shift);
    }
    const int64_t bid = blockIdx.x;
    double acc = 0.0;
#pragma unroll
    for (int s = 0; s < F::R / F::RI; ++s)
        x_c2r_block<T, PLI, F::RI, EPI_ADJOINT, PAD, false, false, true, PRE>(data, nullptr, nrows, tw, lt_shift, sc, ea,
                                                                              bid * (F::R / F::RI) + s, sh + s * F::RI * LD,
                                                                              pk, (int)threadIdx.x, &prei, &acc);
    __syncthreads();  // all staged rows written
#pragma unroll
    for (int s = 0; s < F::R / F::RF; ++s)
        x_r2c_block<T, PLF, F::RF, false, PAD, false, true, PRE>(nullptr, data, nrows, tw, lt_shift, bid * (F::R / F::RF) + s,
                                                                 sh + s * F::RF * LD, pk, (int)threadIdx.x, &pref);
    adj_partial(ea, acc, bid);
}

// Pencils per workgroup of the strided passes: 128-byte rows (16 FP32 / 8 FP64 complex) as long as
// the workgroup's LDS tile stays within 128 KB.
template <typename T, int L>
struct WMax {
    static constexpr int pref = 128 / (int)sizeof(cx<T>);
    static constexpr int cap = (131072 / (L * (int)sizeof(cx<T>))) < 2 ? 2 : (131072 / (L * (int)sizeof(cx<T>)));
    static constexpr int value = pref < cap ? pref : cap;
};

// Tile of the strided passes (y, and the last-axis step) per length: W pencils per workgroup,
// E elements per thread (0: the schedule's largest radix), G LDS groups (fft_stages), state
// prefetch in the step.  Default: WMax pencils, one LDS area.  Long FP32 pencils, measured on
// MI355X: at 1024, 16 pencils with 32 elements per thread and two LDS groups (512 threads, 64 KB:
// two workgroups per CU); at 2048 the same with 1024 threads and 128 KB, which keeps the column
// tile a whole 128-byte line (the default 8 pencils leave 64-byte tiles: y 19.1 -> 15.9 ms and
// z 63 -> 50 ms at 2048^3).
template <typename T, int L>
struct PencilTile {
    static constexpr int W = WMax<T, L>::value, E = 0, G = 1;
    // Lengths with factors 3, 5, 7 load the state after the forward transform: at 375 points and more they
    // hold 15 to 30 elements per thread (750: 20, where 20 more pass the 128 registers that 13 waves per CU
    // allow), and for the shorter ones, of 6 to 20 elements, the prefetch has not been measured.
    static constexpr bool PF = is_pow2c(L);
};
template <>
struct PencilTile<float, 1024> {
    static constexpr int W = 16, E = 32, G = 2;
    static constexpr bool PF = false;
};
template <>
struct PencilTile<float, 1400> {  // 16 pencils of 1400 (800 threads) in two LDS groups (88 KB)
    static constexpr int W = 16, E = 0, G = 2;
    static constexpr bool PF = false;
};
template <>
struct PencilTile<double, 1400> {  // 8 pencils (128-byte tiles) in two LDS groups (88 KB)
    static constexpr int W = 8, E = 0, G = 2;
    static constexpr bool PF = false;
};
template <>
struct PencilTile<float, 2048> {
    static constexpr int W = 16, E = 32, G = 2;  // whole 128-byte lines; 1024 threads, 128 KB
    static constexpr bool PF = false;
};
// Narrow tiles of the strided passes, for launches whose full-width tiles would not fill the chip (the
// launcher's rule, kFillTiles): as many pencils as make one wavefront, at least two (pair tiles are
// split in halves).  A pass over few pencils is bound by the latency of one workgroup's chain of loads,
// exchanges and stores, and most CUs have none: one 512-point tile of 16 pencils per CU puts a 512^2
// step's whole last-axis pass on 16 of 256 CUs.  Narrow tiles read and write parts of a 128-byte line;
// the tiles that share one run on one XCD (xcd_tile_order), and such grids fit the L2s.
template <class PL>
struct NarrowTile {
    static constexpr int W = 64 / PL::Tp < 2 ? 2 : 64 / PL::Tp;
    // four pencils where a launch of them still has a workgroup per CU: more of each line per workgroup
    // (2048^2 FP32: 21.6 against 29.9 us; with fewer workgroups, 1024^2: 13.2 against 12.8)
    static constexpr int W4 = W < 4 && is_pow2c(PL::L) ? 4 : W;
};
// LDS slot of element e: with LP (narrow tiles) one spare slot after every 8.  A pencil's slots are
// then only a few words wide, and the first stage's writes, R elements apart between neighbouring
// threads, would meet on two bank positions.
template <bool LP>
__host__ __device__ constexpr int pencil_slot(int e)
{
    return LP ? e + (e >> 3) : e;
}
template <class PL, int E>
using SpreadIf = std::conditional_t<(E > 0), Spread<PL, (E > 0 ? E : PL::Rmax)>, PL>;

// The tile and the radix schedule of a strided-pass candidate C: a plain schedule takes its
// length's PencilTile; a Tiled candidate (fft_core.hpp) its own, W = SEGB / sizeof(complex).
template <typename T, class C, class = void>
struct TileOf {
    using tile = PencilTile<T, C::L>;
    using plan = C;
};
template <typename T, class C>
struct TileOf<T, C, std::void_t<typename C::plan>> {
    struct tile {
        static constexpr int W = C::seg_bytes / (int)sizeof(cx<T>), E = C::elems, G = C::groups;
        static constexpr bool PF = C::prefetch;
    };
    using plan = typename C::plan;
};

// Schedule PL in the tile of candidate C, as a candidate.
template <class C, class PL, class = void>
struct InitTiled : PL {};
template <class C, class PL>
struct InitTiled<C, PL, std::void_t<typename C::plan>> {
    using plan = PL;
    static constexpr int L = PL::L, seg_bytes = C::seg_bytes, elems = C::elems, groups = C::groups;
    static constexpr bool prefetch = C::prefetch;
};
template <class C, class PL>
using InitTile = std::conditional_t<std::is_same_v<typename PlanOf<C>::type, C>, PL, InitTiled<C, PL>>;

// ------------------------------------------------------------------------------------------------
// Workgroup order for column tiles narrower than a 128-byte line.  Consecutive workgroups are
// dispatched to the 8 XCDs in turn, so workgroups b, b + 8, ..., b + 8 (G - 1) share one XCD and
// its L2; they are given G adjacent tiles, which then share every line in that L2 instead of
// fetching and writing it from G XCDs.  A permutation of [0, n): an incomplete last group keeps
// its indices.
__device__ __forceinline__ int64_t xcd_tile_order(int64_t b, int64_t n, int G)
{
    if (G <= 1) return b;
    const int64_t span = 8 * (int64_t)G, full = n - n % span;
    if (b >= full) return b;
    const int64_t grp = b / span, w = b - grp * span;
    return (grp * 8 + (w & 7)) * G + (w >> 3);
}

// ------------------------------------------------------------------------------------------------
// Strided complex FFT along one axis, out of place or in place (src == dst).
// Pencil (batch, col), col < ncols, has element e = t + k at am.base(batch, col) + am.elem(t) +
// k am.estride (AxisMap in types.hpp; every step k the schedule takes is a multiple of 2^am.ezs, which
// the launcher checks).  A workgroup handles W adjacent columns (W <= WMAX); its threads are laid out
// column-fastest so each load/store instruction moves W * sizeof(cx) contiguous bytes per element
// row (within one 128-byte column chunk).  `bid` is the logical tile index (see xcd_tile_order).
template <typename T, class PL, int WMAX, int DIR, bool NT = false, int G = 1, bool LP = false>
__device__ __forceinline__ void axis_c2c_block(const cx<T> *src, cx<T> *dst, int W, int64_t ncols, const AxisMap &am,
                                               int64_t tiles_per_batch, const cx<T> *__restrict__ tw, int lt_shift,
                                               int64_t bid, cx<T> *sh,
                                               const int tid = (int)threadIdx.x)
{
    constexpr int L = PL::L, Tp = PL::Tp, R0 = PL::first, Rl = PL::last, Rmax = PL::Rmax;
    const int p = tid % WMAX, t = tid / WMAX;
    const int64_t batch = bid / tiles_per_batch, tile = bid - batch * tiles_per_batch;
    const int64_t col = tile * W + p;
    const bool valid = p < W && col < ncols;
    const int64_t base = am.base(batch, valid ? col : 0) + am.elem(t);
    const int64_t estride = am.estride;
    constexpr bool PRE = LP && preload_tw<T, PL>();
    StageTw<T, PL> pre;
    cx<T> v[Rmax];
#pragma unroll
    for (int b = 0; b < PL::nb(R0); ++b)
        if (PL::jok(t + b * Tp, R0))
#pragma unroll
        for (int r = 0; r < R0; ++r)
            v[b * R0 + r] = valid ? ld_grid<NT>(&src[base + (int64_t)(b * Tp + r * (L / R0)) * estride])
                                  : cx<T>{T(0), T(0)};
    constexpr int GW = WMAX / G;  // pencils per LDS group (see fft_stages)
    auto lds = [&](int e) -> cx<T> & { return sh[pencil_slot<LP>(e) * GW + p % GW]; };
    if constexpr (PRE) load_stage_tw<T, PL, TW_STAGE>(pre, t, tw, lt_shift);
    fft_stages<T, PL, DIR, TW_STAGE, G, PRE>(v, t, lds, tw, lt_shift, p / GW, &pre);
    if (valid) {
#pragma unroll
        for (int b = 0; b < PL::nb(Rl); ++b)
            if (PL::jok(t + b * Tp, Rl))
#pragma unroll
            for (int r = 0; r < Rl; ++r)
                st_grid<NT>(&dst[base + (int64_t)(b * Tp + r * (L / Rl)) * estride], v[b * Rl + r]);
    }
}

// Workgroup order: xg >= 1 as xcd_tile_order; xg == 0: workgroup b (on XCD b mod 8) takes the
// batches congruent to b mod 8, their tiles in order, so each XCD works through whole planes (the
// batches past the last multiple of 8 keep the tile order).  Measured for the y pass at 512^3 FP32:
// 188-192 against 206-219 us; at 750^3 (rows not line-aligned, so neighbouring tiles share lines,
// which now meet in one L2) 1.26 against 1.87 ms; slower for the grouped 2048-point tiles.
__device__ __forceinline__ int64_t plane_xcd_order(int64_t b, int64_t tiles_per_batch, int64_t nblocks)
{
    const int64_t batches = nblocks / tiles_per_batch;
    if (b >= (batches - batches % 8) * tiles_per_batch) return b;
    const int64_t k = b >> 3;
    return ((k / tiles_per_batch) * 8 + (b & 7)) * tiles_per_batch + k % tiles_per_batch;
}

// With batch blocks (am.bzs > 0: 2^bzs batches share the rows of one block), the plane order runs
// over whole blocks, and inside a block over tiles first, then the batches of the block, so that
// consecutive workgroups of an XCD read neighbouring 128-byte chunks.
__device__ __forceinline__ int64_t axis_tile(const AxisMap &am, int64_t tiles_per_batch, int xg)
{
    if (xg != 0) return xcd_tile_order(blockIdx.x, gridDim.x, xg);
    const int64_t tb = tiles_per_batch << am.bzs;
    const int64_t u = plane_xcd_order(blockIdx.x, tb, gridDim.x);
    const int64_t sb = u / tb, w = u - sb * tb;
    const int64_t batch = (sb << am.bzs) + (w & ((int64_t(1) << am.bzs) - 1));
    return batch * tiles_per_batch + (w >> am.bzs);
}
template <typename T, class PL, int WMAX, int DIR, int OCC = 1, bool NT = false, int G = 1, bool LP = false>
__global__ __launch_bounds__(WMAX *PL::Tp, OCC) void axis_c2c_kernel(const cx<T> *src, cx<T> *dst, int W,
                                                                 int64_t ncols, AxisMap am, int64_t tiles_per_batch,
                                                                 const cx<T> *__restrict__ tw, int lt_shift, int xg)
{
    static_assert(WMAX % G == 0, "groups of whole pencils");
    __shared__ cx<T> sh[pencil_slot<LP>(PL::L) * WMAX / G];
    const int64_t bid = axis_tile(am, tiles_per_batch, xg);
    axis_c2c_block<T, PL, WMAX, DIR, NT, G, LP>(src, dst, W, ncols, am, tiles_per_batch, tw, lt_shift, bid, sh);
}

// ------------------------------------------------------------------------------------------------
// Last-axis pass (z in 3D, y in 2D): FFT length L = n0 along the slowest axis, rows = n1 (3D) or 1
// (2D), M columns per row.  Element e of pencil (row, kx) sits at e*nrows*M + row*M + kx.
//
// Column kx = 0 pencils need their mirror pencil (row' = -row mod nrows, element -e mod L) to
// separate the two folded planes.  Tiles: W adjacent columns of one row for column tiles >= 1;
// column tile 0 is covered by "pair tiles" that take W/2 columns of row a and the same W/2 columns
// of its mirror row b (pairs (0, nrows/2) and (i, nrows-i)), so a pencil and its mirror always
// share a workgroup.  With nrows == 1 every kx = 0 pencil is its own mirror.
enum { LA_STEP = 0, LA_R2C_NATURAL = 1, LA_C2R_NATURAL = 2, LA_ADJOINT = 3 };

template <typename T>
struct LastAxisArgs {
    const cx<T> *src;  // packed (STEP, R2C_NATURAL, ADJOINT) or natural (C2R_NATURAL) input
    cx<T> *dst;        // packed (STEP, C2R_NATURAL, ADJOINT: mu) or natural (R2C_NATURAL) output
    cx<T> *dst2;       // ADJOINT: nu
    cx<T> *state;      // STEP: native state, updated in place
    int64_t nrows;
    int M;
    int W;
    int tiles_per_row;
    int xg;            // 2D: workgroups per line (xcd_tile_order), 0 or 1 for whole-line tiles
    const cx<T> *tw;
    int lt_shift;
    ModelParams<T> mp;
    Pack pk;   // layout of the packed arrays src, dst, state (natural arrays: rows of M + 1)
    Pack pk2;  // layout of dst2 (ADJOINT's nu: plain rows of M, see x_c2r_block's EPI_ADJOINT)
};

struct SlotInfo {
    int64_t row;
    int kx;
    int partner;  // partner slot for kx == 0 pencils, -1 otherwise
    bool has_pairs;
};

// Order of the workgroups over the column tiles (3D):
//   ORD_TILE: consecutive workgroups take adjacent column tiles of one row (default);
//   ORD_ROW: consecutive workgroups take consecutive rows of one column tile (measured slightly
//            slower at 512^3);
//   ORD_XCD_ROW: workgroup b runs on XCD b mod 8 (round-robin dispatch); each XCD takes whole rows
//            (rows r with r mod 8 = its XCD, tiles in order), so that tiles whose rows are not
//            line-aligned (natural half spectrum, pitch M + 1) share their boundary lines in one
//            L2; rows past the last multiple of 8 keep the ORD_TILE order.  Used by the step's fused
//            pass too, where it measured 1.5-2 % faster than ORD_TILE (512^3 and 2048^3 FP32).
// IL: in the pair tiles, slots alternate between the two rows (slot p and its mirror p ^ 1 hold the
// same column), so that a pencil and its mirror stay in one group of adjacent slots; otherwise the
// first W/2 slots hold row k_y and the others row -k_y.
enum { ORD_TILE = 0, ORD_ROW = 1, ORD_XCD_ROW = 2 };
template <int ORD = ORD_TILE, bool IL = false>
__device__ __forceinline__ SlotInfo la_slot(int64_t nrows, int TR, int W, int p, int64_t bid)
{
    SlotInfo s;
    if (nrows == 1) {
        s.row = 0;
        s.kx = (int)bid * W + p;
        s.partner = (s.kx == 0) ? p : -1;
        s.has_pairs = (bid == 0);
        return s;
    }
    const int64_t n_normal = nrows * (TR - 1);
    if (bid < n_normal) {
        if (ORD == ORD_ROW) {
            s.row = bid % nrows;
            s.kx = (int)(1 + bid / nrows) * W + p;
        } else if (ORD == ORD_XCD_ROW && bid < (nrows - (nrows & 7)) * (TR - 1)) {
            const int64_t k = bid >> 3;
            s.row = (k / (TR - 1)) * 8 + (bid & 7);
            s.kx = (int)(1 + k % (TR - 1)) * W + p;
        } else {
            s.row = bid / (TR - 1);
            s.kx = (int)(1 + bid % (TR - 1)) * W + p;
        }
        s.partner = -1;
        s.has_pairs = false;
        return s;
    }
    // pair tiles: k in [0, nrows) takes pair i (rows i and -i; i = 0: rows 0 and nrows / 2) and half
    // h of column tile 0.  In whole groups of 16 the two halves of a pair are 8 apart (k and k + 8
    // run on one XCD under round-robin dispatch), so the lines they share meet in one L2 instead of
    // being fetched by two XCDs; a last incomplete group takes the halves in turn.
    const int64_t k = bid - n_normal, full = nrows - nrows % 16;
    const int64_t i = k < full ? ((k >> 4) << 3) + (k & 7) : (k >> 1);
    const int h = (int)(k < full ? ((k >> 3) & 1) : (k & 1)), hw = W >> 1;
    const int64_t ra = (i == 0) ? 0 : i, rb = (i == 0) ? nrows / 2 : nrows - i;
    if constexpr (IL) {
        const bool first = (p & 1) == 0;
        s.row = first ? ra : rb;
        s.kx = h * hw + (p >> 1);
        s.partner = (s.kx == 0) ? ((i == 0) ? p : (p ^ 1)) : -1;
    } else {
        const bool first = p < hw;
        s.row = first ? ra : rb;
        s.kx = h * hw + (first ? p : p - hw);
        s.partner = (s.kx == 0) ? ((i == 0) ? p : (first ? p + hw : p - hw)) : -1;
    }
    s.has_pairs = (h == 0);
    return s;
}

// Order of the pair tiles of la_slot where they are all there is (rows of at most W columns): the G tiles that
// share the lines of neighbouring rows run on one XCD (xcd_tile_order).  The tile of pair i and half h in
// the place that la_slot gives it.
__device__ __forceinline__ int64_t la_pair_order(int64_t bid, int64_t nrows, int G)
{
    const int64_t u = xcd_tile_order(bid, nrows, G), i = u >> 1, h = u & 1;
    return u < nrows - nrows % 16 ? ((i >> 3) << 4) + (h << 3) + (i & 7) : u;
}

// G > 1 (STEP only): the pencils form G groups of WMAX / G adjacent slots that take turns in an LDS
// area of L * WMAX / G values (see fft_stages); pair tiles then interleave their two rows.
template <typename T, class PL, int WMAX, int MODE, bool PF = true, int ORD = ORD_TILE, bool NT = false, int G = 1,
          bool LP = false>
__device__ __forceinline__ void last_axis_block(const LastAxisArgs<T> &a, int64_t bid, cx<T> *sh)
{
    static_assert(G == 1 || MODE == LA_STEP, "grouped LDS only in the step");
    static_assert(WMAX % G == 0 && (G == 1 || (WMAX / G) % 2 == 0), "groups must hold whole pairs");
    constexpr int L = PL::L, Tp = PL::Tp, Rmax = PL::Rmax, GW = WMAX / G;
    constexpr bool IL = G > 1;
    using PR = typename PL::Reverse;  // inverse schedule: its first radix is PL's last
    constexpr int Rl = PL::last;
    const int tid = threadIdx.x, p = tid % WMAX, t = tid / WMAX, grp = p / GW;
    const int W = a.W;
    const int64_t nrows = a.nrows, M = a.M;
    const SlotInfo si = la_slot<ORD, IL>(nrows, a.tiles_per_row, W, p < W ? p : 0, bid);
    const bool valid = p < W && si.kx < M;  // the last column tile of a row may be partial
    auto lds = [&](int e) -> cx<T> & { return sh[pencil_slot<LP>(e) * GW + p % GW]; };
    // Element e = t + k of this lane's pencil in a packed array lies at pk.at(t, row, kx) + k estride
    // (k a multiple of the layout's block size Z, which the launcher checks).  The address is split
    // into a wave-uniform part (the tile origin, the wave's first t, and k * estride: scalar
    // registers) and a per-lane 32-bit byte offset, so no per-element 64-bit vector arithmetic is
    // needed.
    const Pack &pk = a.pk;
    const int64_t estride = pk.e_stride();
    const SlotInfo s0 = la_slot<ORD, IL>(nrows, a.tiles_per_row, W, 0, bid);
    const int t0 = __builtin_amdgcn_readfirstlane(t);
    const int64_t uoff = pk.at(t0, s0.row, s0.kx);
    const uint32_t loff = (uint32_t)((pk.at(t, si.row, si.kx) - uoff) * (int64_t)sizeof(cx<T>));
    auto gp = [&](const cx<T> *base, int k) -> cx<T> * {
        return reinterpret_cast<cx<T> *>(
            reinterpret_cast<char *>(const_cast<cx<T> *>(base) + uoff + (int64_t)k * estride) + loff);
    };
    const ModelParams<T> &mp = a.mp;
    const T ky = mp.fk[1] * (T)signed_index(si.row, nrows);
    const T kx = mp.fk[2] * (T)si.kx;
    const T kxn = mp.fk[2] * (T)M;  // x Nyquist wavenumber
    cx<T> v[Rmax];

    if constexpr (MODE == LA_C2R_NATURAL) {
        // natural half spectrum in: fold kx = 0 and kx = M (projected) into one plane, inverse FFT
        constexpr int R0 = PR::first;
        const int64_t prow =
            (si.partner >= 0) ? la_slot<ORD>(nrows, a.tiles_per_row, W, si.partner, bid).row : 0;
        const int64_t pitch = M + 1;
#pragma unroll
        for (int b = 0; b < PL::nb(R0); ++b)
            if (PL::jok(t + b * Tp, R0))
#pragma unroll
            for (int r = 0; r < R0; ++r) {
                const int e = t + b * Tp + r * (L / R0);
                cx<T> z = {T(0), T(0)};
                if (valid) {
                    const int64_t i0 = ((int64_t)e * nrows + si.row) * pitch;
                    if (si.partner < 0) {
                        z = a.src[i0 + si.kx];
                    } else {
                        const int ep = neg_mod<L>(e);
                        const int64_t i1 = ((int64_t)ep * nrows + prow) * pitch;
                        const cx<T> x0 = a.src[i0], x0p = a.src[i1], xn = a.src[i0 + M], xnp = a.src[i1 + M];
                        const T h = T(0.5);
                        const cx<T> P0 = {(x0.x + x0p.x) * h, (x0.y - x0p.y) * h};
                        const cx<T> PN = {(xn.x + xnp.x) * h, (xn.y - xnp.y) * h};
                        z = {P0.x - PN.y, P0.y + PN.x};
                    }
                }
                v[b * R0 + r] = z;
            }
        fft_stages<T, PR, +1>(v, t, lds, a.tw, a.lt_shift);
        if (valid) {
            constexpr int Rf = PR::last;
#pragma unroll
            for (int b = 0; b < PL::nb(Rf); ++b)
                if (PL::jok(t + b * Tp, Rf))
#pragma unroll
                for (int r = 0; r < Rf; ++r) st_grid<NT>(gp(a.dst, b * Tp + r * (L / Rf)), v[b * Rf + r]);
        }
        return;
    } else {
        // STEP with PF: the state values this thread updates are loaded before the forward FFT so
        // that their latency overlaps the FFT
        constexpr bool PRE = LP && preload_tw<T, PL>();
        constexpr bool SYM = std::is_same_v<PL, PR>;  // one set of twiddles serves both directions
        StageTw<T, PL> pre;
        StageTw<T, PR> prei;
        cx<T> spre[(MODE == LA_STEP && PF) ? Rmax : 1];
        if constexpr (MODE == LA_STEP && PF) {
#pragma unroll
            for (int b = 0; b < PL::nb(Rl); ++b)
                if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                for (int r = 0; r < Rl; ++r)
                    spre[b * Rl + r] = valid ? ld_grid<NT>(gp(a.state, b * Tp + r * (L / Rl))) : cx<T>{T(0), T(0)};
        }
        // packed input, forward FFT
        constexpr int R0 = PL::first;
#pragma unroll
        for (int b = 0; b < PL::nb(R0); ++b)
            if (PL::jok(t + b * Tp, R0))
#pragma unroll
            for (int r = 0; r < R0; ++r)
                v[b * R0 + r] = valid ? ld_grid<NT>(gp(a.src, b * Tp + r * (L / R0))) : cx<T>{T(0), T(0)};
        if constexpr (PRE) {
            load_stage_tw<T, PL, TW_STAGE>(pre, t, a.tw, a.lt_shift);
            if constexpr (!SYM && MODE == LA_STEP) load_stage_tw<T, PR, TW_STAGE>(prei, t, a.tw, a.lt_shift);
        }
        fft_stages<T, PL, -1, TW_STAGE, G, PRE>(v, t, lds, a.tw, a.lt_shift, grp, &pre);
        // forward spectrum in natural order: v[b*Rl + r] = X(e), e = t + b*Tp + r*L/Rl
        auto partner_val = [&](int e) -> cx<T> { return sh[pencil_slot<LP>(neg_mod<L>(e)) * GW + si.partner % GW]; };
        auto spectrum_to_lds = [&]() {
#pragma unroll
            for (int b = 0; b < PL::nb(Rl); ++b)
                if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                for (int r = 0; r < Rl; ++r) lds(t + b * Tp + r * (L / Rl)) = v[b * Rl + r];
        };

        if constexpr (MODE == LA_R2C_NATURAL || MODE == LA_ADJOINT) {
            if (si.has_pairs) {  // uniform per workgroup
                __syncthreads();
                spectrum_to_lds();
                __syncthreads();
            }
        }
        if constexpr (MODE == LA_R2C_NATURAL) {
            const int64_t pitch = M + 1;
            if (valid) {
#pragma unroll
                for (int b = 0; b < PL::nb(Rl); ++b)
                    if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                    for (int r = 0; r < Rl; ++r) {
                        const int e = t + b * Tp + r * (L / Rl);
                        const int64_t i0 = ((int64_t)e * nrows + si.row) * pitch;
                        const cx<T> z = v[b * Rl + r];
                        if (si.partner < 0) {
                            a.dst[i0 + si.kx] = z;
                        } else {
                            const cx<T> zp = partner_val(e);
                            const T h = T(0.5);
                            a.dst[i0] = {(z.x + zp.x) * h, (z.y - zp.y) * h};
                            a.dst[i0 + M] = {(z.y + zp.y) * h, (zp.x - z.x) * h};
                        }
                    }
            }
            return;
        } else if constexpr (MODE == LA_STEP) {
            // Semi-implicit update.  Pencils off the folded column: S <- (S - dt q N) A(q).  Folded
            // column: the two planes X0 (q0) and XN (qN) are separated with the mirror element -k,
            // which another thread owns; the mirror's N comes from LDS now, its S in a second LDS
            // round, so no thread reads a state value that another thread has already updated.
            const T dt = mp.dt, nl = mp.nl, h = T(0.5);
            // narrow tiles: the mirror's S goes through an LDS area of its own in the round of N, behind
            // the tile's slots (fold_slots)
            constexpr bool ONE = LP && PF;
            cx<T> *const sh2 = sh + pencil_slot<LP>(L) * GW;
            auto fold = [&](int q) { return nrows == 1 || q == 0 ? 0 : 1; };  // folded pencil in slot q
            if constexpr (ONE) {
                if (si.has_pairs) {  // uniform per workgroup
                    __syncthreads();
                    if (si.partner >= 0 && valid) {  // (slots past W repeat slot 0)
#pragma unroll
                        for (int b = 0; b < PL::nb(Rl); ++b)
                            if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                            for (int r = 0; r < Rl; ++r) {
                                const int e = t + b * Tp + r * (L / Rl);
                                lds(e) = v[b * Rl + r];
                                sh2[fold(p) * L + e] = spre[b * Rl + r];
                            }
                    }
                    __syncthreads();
                }
            } else if (si.has_pairs) {  // uniform per workgroup
#pragma unroll
                for (int gg = 0; gg < G; ++gg) {
                    const bool mine = (G == 1) || (grp == gg);
                    __syncthreads();
                    if (mine) spectrum_to_lds();
                    __syncthreads();
                    if (mine && si.partner >= 0) {
#pragma unroll
                        for (int b = 0; b < PL::nb(Rl); ++b)
                            if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                            for (int r = 0; r < Rl; ++r) {
                                const int e = t + b * Tp + r * (L / Rl);
                                const T kz = mp.fk[0] * (T)signed_index(e, L);
                                const cx<T> N = {v[b * Rl + r].x * nl, v[b * Rl + r].y * nl};
                                const cx<T> Np = {partner_val(e).x * nl, partner_val(e).y * nl};
                                const cx<T> N0 = {(N.x + Np.x) * h, (N.y - Np.y) * h};
                                const cx<T> NN = {(N.y + Np.y) * h, (Np.x - N.x) * h};
                                const T q0 = kz * kz + ky * ky, qn = q0 + kxn * kxn;
                                const T g0 = dt * q0 * amult(mp, q0), gn = dt * qn * amult(mp, qn);
                                // G = -(g0 N0 + i gn NN): the cubic term's share of the new value
                                v[b * Rl + r] = {-g0 * N0.x + gn * NN.y, -g0 * N0.y - gn * NN.x};
                            }
                    }
                }
            }
            if (si.partner < 0) {
#pragma unroll
                for (int b = 0; b < PL::nb(Rl); ++b)
                    if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                    for (int r = 0; r < Rl; ++r) {
                        const int e = t + b * Tp + r * (L / Rl);
                        const T kz = mp.fk[0] * (T)signed_index(e, L);
                        const cx<T> N = {v[b * Rl + r].x * nl, v[b * Rl + r].y * nl};
                        cx<T> *gi = gp(a.state, b * Tp + r * (L / Rl));
                        cx<T> S;
                        if constexpr (PF)
                            S = spre[b * Rl + r];
                        else
                            S = valid ? ld_grid<NT>(gi) : cx<T>{T(0), T(0)};
                        const T q = kz * kz + ky * ky + kx * kx;
                        const T A = amult(mp, q), dq = dt * q;
                        const cx<T> Snew = {(S.x - dq * N.x) * A, (S.y - dq * N.y) * A};
                        if (valid) st_grid<NT>(gi, Snew);
                        v[b * Rl + r] = Snew;
                    }
            }
            if constexpr (ONE) {
                if (si.partner >= 0) {
#pragma unroll
                    for (int b = 0; b < PL::nb(Rl); ++b)
                        if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                        for (int r = 0; r < Rl; ++r) {
                            const int e = t + b * Tp + r * (L / Rl);
                            const T kz = mp.fk[0] * (T)signed_index(e, L);
                            const T q0 = kz * kz + ky * ky, qn = q0 + kxn * kxn;
                            const T A0 = amult(mp, q0), AN = amult(mp, qn);
                            // the operations of the two rounds below, in their order
                            const cx<T> Nr = partner_val(e), Sp = sh2[fold(si.partner) * L + neg_mod<L>(e)];
                            const cx<T> N = {v[b * Rl + r].x * nl, v[b * Rl + r].y * nl}, S = spre[b * Rl + r];
                            const cx<T> Np = {Nr.x * nl, Nr.y * nl};
                            const cx<T> N0 = {(N.x + Np.x) * h, (N.y - Np.y) * h};
                            const cx<T> NN = {(N.y + Np.y) * h, (Np.x - N.x) * h};
                            const T g0 = dt * q0 * A0, gn = dt * qn * AN;
                            const cx<T> Gt = {-g0 * N0.x + gn * NN.y, -g0 * N0.y - gn * NN.x};
                            const cx<T> S0 = {(S.x + Sp.x) * h, (S.y - Sp.y) * h};
                            const cx<T> SN = {(S.y + Sp.y) * h, (Sp.x - S.x) * h};
                            const cx<T> Snew = {A0 * S0.x - AN * SN.y + Gt.x, A0 * S0.y + AN * SN.x + Gt.y};
                            if (valid) st_grid<NT>(gp(a.state, b * Tp + r * (L / Rl)), Snew);
                            v[b * Rl + r] = Snew;
                        }
                }
            } else if (si.has_pairs) {  // uniform per workgroup
#pragma unroll
                for (int gg = 0; gg < G; ++gg) {
                    const bool mine = (G == 1) || (grp == gg);
                    __syncthreads();  // every mirror N has been read
                    if (mine && si.partner >= 0 && valid) {
#pragma unroll
                        for (int b = 0; b < PL::nb(Rl); ++b)
                            if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                            for (int r = 0; r < Rl; ++r) {
                                const int e = t + b * Tp + r * (L / Rl);
                                if constexpr (PF)
                                    lds(e) = spre[b * Rl + r];
                                else
                                    lds(e) = ld_grid<NT>(gp(a.state, b * Tp + r * (L / Rl)));
                            }
                    }
                    __syncthreads();
                    if (mine && si.partner >= 0) {
#pragma unroll
                        for (int b = 0; b < PL::nb(Rl); ++b)
                            if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                            for (int r = 0; r < Rl; ++r) {
                                const int e = t + b * Tp + r * (L / Rl);
                                const T kz = mp.fk[0] * (T)signed_index(e, L);
                                cx<T> *gi = gp(a.state, b * Tp + r * (L / Rl));
                                cx<T> S;
                                if constexpr (PF)
                                    S = spre[b * Rl + r];
                                else
                                    S = valid ? ld_grid<NT>(gi) : cx<T>{T(0), T(0)};
                                const cx<T> Sp = partner_val(e);
                                const cx<T> S0 = {(S.x + Sp.x) * h, (S.y - Sp.y) * h};
                                const cx<T> SN = {(S.y + Sp.y) * h, (Sp.x - S.x) * h};
                                const T q0 = kz * kz + ky * ky, qn = q0 + kxn * kxn;
                                const T A0 = amult(mp, q0), AN = amult(mp, qn);
                                const cx<T> Gt = v[b * Rl + r];
                                // A0 S0 + i AN SN + G
                                const cx<T> Snew = {A0 * S0.x - AN * SN.y + Gt.x, A0 * S0.y + AN * SN.x + Gt.y};
                                if (valid) st_grid<NT>(gi, Snew);
                                v[b * Rl + r] = Snew;
                            }
                    }
                }
            }
            if constexpr (PRE && SYM)
                fft_stages<T, PR, +1, TW_STAGE, G, true>(v, t, lds, a.tw, a.lt_shift, grp, &pre);
            else
                fft_stages<T, PR, +1, TW_STAGE, G, PRE>(v, t, lds, a.tw, a.lt_shift, grp, &prei);
            if (valid) {
                constexpr int Rf = PR::last;
#pragma unroll
                for (int b = 0; b < PL::nb(Rf); ++b)
                    if (PL::jok(t + b * Tp, Rf))
#pragma unroll
                    for (int r = 0; r < Rf; ++r) st_grid<NT>(gp(a.dst, b * Tp + r * (L / Rf)), v[b * Rf + r]);
            }
        } else if constexpr (MODE == LA_ADJOINT) {
            cx<T> w[Rmax];
#pragma unroll
            for (int b = 0; b < PL::nb(Rl); ++b)
                if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                for (int r = 0; r < Rl; ++r) {
                    const int e = t + b * Tp + r * (L / Rl);
                    const T kz = mp.fk[0] * (T)signed_index(e, L);
                    const cx<T> z = v[b * Rl + r];
                    cx<T> mu, nu;
                    if (si.partner < 0) {
                        const T q = kz * kz + ky * ky + kx * kx;
                        const T A = amult(mp, q);
                        mu = {z.x * A, z.y * A};
                        nu = {mu.x * q, mu.y * q};
                    } else {
                        const cx<T> zp = partner_val(e);
                        const T h = T(0.5);
                        const cx<T> U = {(z.x + zp.x) * h, (z.y - zp.y) * h};
                        const cx<T> V = {(z.y + zp.y) * h, (zp.x - z.x) * h};
                        const T q0 = kz * kz + ky * ky, qn = q0 + kxn * kxn;
                        const T A0 = amult(mp, q0), AN = amult(mp, qn);
                        const cx<T> mU = {U.x * A0, U.y * A0}, mV = {V.x * AN, V.y * AN};
                        mu = {mU.x - mV.y, mU.y + mV.x};
                        nu = {mU.x * q0 - mV.y * qn, mU.y * q0 + mV.x * qn};
                    }
                    v[b * Rl + r] = mu;
                    w[b * Rl + r] = nu;
                }
            constexpr int Rf = PR::last;
            const int64_t uoff2 = a.pk2.at(t0, s0.row, s0.kx), estride2 = a.pk2.e_stride();
            const uint32_t loff2 = (uint32_t)((a.pk2.at(t, si.row, si.kx) - uoff2) * (int64_t)sizeof(cx<T>));
            auto gp2 = [&](cx<T> *base, int k) -> cx<T> * {
                return reinterpret_cast<cx<T> *>(reinterpret_cast<char *>(base + uoff2 + (int64_t)k * estride2) + loff2);
            };
            fft_stages<T, PR, +1>(v, t, lds, a.tw, a.lt_shift);
            if (valid) {
#pragma unroll
                for (int b = 0; b < PL::nb(Rf); ++b)
                    if (PL::jok(t + b * Tp, Rf))
#pragma unroll
                    for (int r = 0; r < Rf; ++r) *gp(a.dst, b * Tp + r * (L / Rf)) = v[b * Rf + r];
            }
            fft_stages<T, PR, +1>(w, t, lds, a.tw, a.lt_shift);
            if (valid) {
#pragma unroll
                for (int b = 0; b < PL::nb(Rf); ++b)
                    if (PL::jok(t + b * Tp, Rf))
#pragma unroll
                    for (int r = 0; r < Rf; ++r) *gp2(a.dst2, b * Tp + r * (L / Rf)) = w[b * Rf + r];
            }
        }
    }
}

template <typename T, class PL, int WMAX, int MODE, int OCC = 1, bool PF = true, int ORD = ORD_TILE, bool NT = false,
          int G = 1, bool LP = false>
__global__ __launch_bounds__(WMAX *PL::Tp, OCC) void last_axis_kernel(LastAxisArgs<T> a)
{
    // narrow step tiles: two folded pencils' state values behind the tile's slots
    constexpr int fold_slots = (LP && PF && MODE == LA_STEP) ? 2 * PL::L : 0;
    __shared__ cx<T> sh[pencil_slot<LP>(PL::L) * WMAX / G + fold_slots];
    const int64_t bid = LP && a.nrows == 1 ? xcd_tile_order(blockIdx.x, gridDim.x, a.xg) : blockIdx.x;
    last_axis_block<T, PL, WMAX, MODE, PF, ORD, NT, G, LP>(a, bid, sh);
}

// ------------------------------------------------------------------------------------------------
// Last axis of the 3D r2c into the natural half spectrum (rows of M + 1 values), by line-aligned
// chunks.  The output plane (nrows rows of M + 1) is cut into chunks of C = 128 / sizeof(cx)
// consecutive values; workgroup c owns output positions f = cC .. cC + C - 1 of every plane, i.e.
// one whole 128-byte line per plane (requires nrows (M + 1) % C == 0 and M >= C), so no line is
// written by two workgroups.  Slot p computes the pencil of position f: row f / (M + 1), column
// kx = f % (M + 1).  For 1 <= kx < M that is packed column kx; kx = 0 and kx = M are the two planes
// folded into packed column 0, separated with the mirror pencil (row -k_y, element -k_z), which a
// second round transforms: X0 = (Z(k) + conj Z(-k)) / 2, XM = -i (Z(k) - conj Z(-k)) / 2.  A chunk
// holds at most two such slots; the second round runs only in chunks that have one.  The reads of
// packed columns are not line-aligned; chunks that share input lines run on one XCD.
template <typename T, class PL, int C, int G, bool NT = false>
__global__ __launch_bounds__(C *PL::Tp) void r2c_natural_chunk_kernel(const cx<T> *__restrict__ src,
                                                                      cx<T> *__restrict__ dst, int64_t nrows, int M,
                                                                      const cx<T> *__restrict__ tw, int lt_shift,
                                                                      Pack pk)
{
    constexpr int L = PL::L, Tp = PL::Tp, Rmax = PL::Rmax, R0 = PL::first, Rl = PL::last, GW = C / G;
    __shared__ cx<T> sh[L * GW];
    const int tid = threadIdx.x, p = tid % C, t = tid / C, grp = p / GW;
    auto lds = [&](int e) -> cx<T> & { return sh[e * GW + p % GW]; };
    const int64_t pitch = (int64_t)M + 1, plane = nrows * pitch, nchunks = plane / C;
    const int64_t chunk = xcd_tile_order(blockIdx.x, nchunks, 16);
    const int64_t f = chunk * C + p;
    const int64_t row = f / pitch;
    const int kx = (int)(f - row * pitch);
    const bool fold = (kx == 0 || kx == M);
    const int64_t estride = pk.e_stride();  // element steps k below are multiples of the layout's block
    cx<T> v[Rmax];
    // first sweep: own pencil (folded slots: packed column 0 of this row)
    {
        const cx<T> *col = src + pk.at(t, row, fold ? 0 : kx);
#pragma unroll
        for (int b = 0; b < PL::nb(R0); ++b)
            if (PL::jok(t + b * Tp, R0))
#pragma unroll
            for (int r = 0; r < R0; ++r) v[b * R0 + r] = col[(int64_t)(b * Tp + r * (L / R0)) * estride];
    }
    fft_stages<T, PL, -1, TW_STAGE, G>(v, t, lds, tw, lt_shift, grp);
    if (!fold) {
#pragma unroll
        for (int b = 0; b < PL::nb(Rl); ++b)
            if (PL::jok(t + b * Tp, Rl))
#pragma unroll
            for (int r = 0; r < Rl; ++r) st_grid<NT>(&dst[(int64_t)(t + b * Tp + r * (L / Rl)) * plane + f], v[b * Rl + r]);
    }
    if (!__syncthreads_or(fold)) return;  // uniform: the chunk has no folded slot
    // second sweep: mirror pencils of the folded slots
    cx<T> z[Rmax];
#pragma unroll
    for (int i = 0; i < Rmax; ++i) z[i] = v[i];
    {
        const int64_t mrow = (nrows - row) % nrows;
        const cx<T> *col = src + pk.at(t, mrow, 0);
#pragma unroll
        for (int b = 0; b < PL::nb(R0); ++b)
            if (PL::jok(t + b * Tp, R0))
#pragma unroll
            for (int r = 0; r < R0; ++r)
                v[b * R0 + r] = fold ? col[(int64_t)(b * Tp + r * (L / R0)) * estride] : cx<T>{T(0), T(0)};
    }
    fft_stages<T, PL, -1, TW_STAGE, G>(v, t, lds, tw, lt_shift, grp);
    const T h = T(0.5);
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
        const bool mine = (G == 1) || (grp == gg);
        __syncthreads();
        if (mine) {
#pragma unroll
            for (int b = 0; b < PL::nb(Rl); ++b)
                if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                for (int r = 0; r < Rl; ++r) lds(t + b * Tp + r * (L / Rl)) = v[b * Rl + r];
        }
        __syncthreads();
        if (mine && fold) {
#pragma unroll
            for (int b = 0; b < PL::nb(Rl); ++b)
                if (PL::jok(t + b * Tp, Rl))
#pragma unroll
                for (int r = 0; r < Rl; ++r) {
                    const int e = t + b * Tp + r * (L / Rl);
                    const cx<T> a = z[b * Rl + r], m = lds(neg_mod<L>(e));
                    const cx<T> out = (kx == 0) ? cx<T>{(a.x + m.x) * h, (a.y - m.y) * h}
                                                : cx<T>{(a.y + m.y) * h, (m.x - a.x) * h};
                    st_grid<NT>(&dst[(int64_t)e * plane + f], out);
                }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Reductions (FP64 accumulation, fixed grid and order: deterministic).

// The passes below read whole grids once and are bound by HBM bandwidth, so what matters is bytes in
// flight: a thread issues its loads in groups (four 16-byte loads, or four modes of a row) before it
// uses the first.  Measured with scalar loads and 64-bit divisions per mode, then in this form,
// 256^3 FP32: sum 21 -> 12 us (5.5 TB/s), energy 52 + 22 -> 33 us (one launch, 4.1 TB/s), export 35 ->
// 25 us (5.4 TB/s).  The final sums over the block partials are a chain of load latencies in one
// thread, so a workgroup shares them: mass 58 -> 4 us, energy 112 -> 5 us.

// Adds f(x[i]) over a grid-stride range of n values, block `blk` of `nblk`; x 16-byte aligned.
template <typename T, class F>
__device__ __forceinline__ double stream_sum(const T *__restrict__ x, int64_t n, int64_t blk, int64_t nblk, F &&f)
{
    constexpr int V = 16 / (int)sizeof(T), U = 4;
    typedef T vec __attribute__((ext_vector_type(V)));
    const vec *xv = reinterpret_cast<const vec *>(x);
    const int64_t nv = n / V, step = nblk * blockDim.x;
    double acc[U] = {};
    for (int64_t i = blk * blockDim.x + threadIdx.x; i < nv; i += U * step) {
        vec v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = i + u * step < nv ? xv[i + u * step] : vec(T(0));
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < V; ++k) acc[u] += f(v[u][k]);
    }
    const int64_t tail = nv * V + blk * blockDim.x + threadIdx.x;
    if (tail < n) acc[0] += f(x[tail]);
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// Calls f(e, row, kx, s) for every mode of a packed spectrum, s its value: groups of 2^tps threads
// take whole rows (one 32-bit division per row), each thread four modes at a time.
template <typename T, class F>
__device__ __forceinline__ void for_modes(const cx<T> *__restrict__ state, int64_t L, int64_t nrows, int64_t M, int tps,
                                          const Pack &pk, int64_t blk, int64_t nblk, F &&f)
{
    constexpr int U = 4;
    const int tpr = 1 << tps, rows = (int)(L * nrows), stride = (int)(nblk * (blockDim.x >> tps));
    for (int r = (int)(blk * (blockDim.x >> tps)) + (int)(threadIdx.x >> tps); r < rows; r += stride) {
        const int e = (int)((unsigned)r / (unsigned)nrows), row = r - e * (int)nrows;
        const cx<T> *src = state + pk.row_base(e, row);
        for (int k = (int)(threadIdx.x & (unsigned)(tpr - 1)); k < M; k += U * tpr) {
            cx<T> v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = k + u * tpr < M ? src[pk.col(k + u * tpr)] : cx<T>{T(0), T(0)};
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k + u * tpr < M) f(e, row, k + u * tpr, v[u]);
        }
    }
}

// partial[block] = sum of x over a grid-stride range.
template <typename T>
__global__ __launch_bounds__(256) void sum_kernel(const T *__restrict__ x, int64_t n, double *partial)
{
    const double acc = stream_sum(x, n, blockIdx.x, gridDim.x, [](T v) { return (double)v; });
    __shared__ double red[4];
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Sum of partial[0..np) by one workgroup, valid in thread 0 (fixed order for a given np and
// workgroup size).  red: >= blockDim.x / 64 doubles of LDS.
__device__ __forceinline__ double partial_sum(const double *partial, int np, double *red)
{
    double acc = 0.0;
    for (int i = threadIdx.x; i < np; i += blockDim.x) acc += partial[i];
    return block_sum(acc, red);
}

// state[0].x = (T) sum(partial[0..np)) -- the mass mode from an FP64 sum of the field.
template <typename T>
__global__ __launch_bounds__(256) void set_mass_kernel(const double *partial, int np, cx<T> *state)
{
    __shared__ double red[4];
    const double s = partial_sum(partial, np, red);
    if (threadIdx.x == 0) state[0].x = (T)s;
}

// *acc += coef * sum(partial[0..np))
__global__ void accumulate_kernel(const double *partial, int np, double coef, double *acc);

// Partial sums of the energy (FP64 throughout): the first np workgroups the spectral quadratic part,
// sum over the full spectrum of (r + L(q)) |psi_hat|^2 from the native state (geometry as in the
// last-axis pass), into partial[0..np); the next np the quartic part, sum of psi^4 / 4, into
// partial[np..2np).
template <typename T>
__global__ __launch_bounds__(256) void energy_kernel(const cx<T> *__restrict__ state, const T *__restrict__ psi,
                                                     int64_t L, int64_t nrows, int64_t M, int tps, double fk0, double fk1,
                                                     double fk2, double r, double q1sq, double R1, int model, int np,
                                                     double *partial, Pack pk)
{
    auto corr = [&](double q) {
        double a = (1.0 - q) * (1.0 - q);
        if (model == 0) return a;
        double b = q1sq - q;
        return a * (b * b + R1);
    };
    double acc = 0.0;
    if ((int)blockIdx.x < np) {
        for_modes(state, L, nrows, M, tps, pk, blockIdx.x, np, [&](int e, int row, int kx, cx<T> s) {
            const double kz = fk0 * signed_index(e, L), ky = fk1 * signed_index(row, nrows);
            if (kx != 0) {
                const double k = fk2 * (double)kx, q = kz * kz + ky * ky + k * k;
                acc += 2.0 * (r + corr(q)) * ((double)s.x * s.x + (double)s.y * s.y);
            } else {
                const int64_t ep = e == 0 ? 0 : L - e, rp = row == 0 ? 0 : nrows - row;
                const cx<T> sp = state[pk.at(ep, rp, 0)];
                const double ax = 0.5 * ((double)s.x + sp.x), ay = 0.5 * ((double)s.y - sp.y);
                const double bx = 0.5 * ((double)s.y + sp.y), by = 0.5 * ((double)sp.x - s.x);
                const double q0 = kz * kz + ky * ky, kn = fk2 * (double)M, qn = q0 + kn * kn;
                acc += (r + corr(q0)) * (ax * ax + ay * ay) + (r + corr(qn)) * (bx * bx + by * by);
            }
        });
    } else {
        acc = stream_sum(psi, 2 * M * L * nrows, blockIdx.x - np, np, [](T p) {
            const double v = (double)p * (double)p;
            return 0.25 * v * v;
        });
    }
    __shared__ double red[4];
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// out[0] = dV (sum(ps)/(2N) + sum(pq)), out[1] = state[0].x / N.
template <typename T>
__global__ __launch_bounds__(256) void energy_final_kernel(const double *ps, const double *pq, int np, double dV,
                                                           double ntot, const cx<T> *state, double *out)
{
    __shared__ double red[4];
    const double a = partial_sum(ps, np, red);
    const double b = partial_sum(pq, np, red);
    if (threadIdx.x == 0) {
        out[0] = dV * (a / (2.0 * ntot) + b);
        out[1] = (double)state[0].x / ntot;
    }
}

// Native state -> natural half spectrum [L][nrows][M+1].  The thread of a row's folded column writes
// both of its planes, kx = 0 and kx = M.
template <typename T>
__global__ __launch_bounds__(256) void export_kernel(const cx<T> *__restrict__ state, cx<T> *__restrict__ out,
                                                     int64_t L, int64_t nrows, int64_t M, int tps, Pack pk)
{
    for_modes(state, L, nrows, M, tps, pk, blockIdx.x, gridDim.x, [&](int e, int row, int kx, cx<T> s) {
        cx<T> *dst = out + ((int64_t)e * nrows + row) * (M + 1);
        if (kx != 0) {
            dst[kx] = s;
        } else {
            const cx<T> sp = state[pk.at(e == 0 ? 0 : L - e, row == 0 ? 0 : nrows - row, 0)];
            const T h = T(0.5);
            dst[0] = {(s.x + sp.x) * h, (s.y - sp.y) * h};
            dst[M] = {(s.y + sp.y) * h, (sp.x - s.x) * h};
        }
    });
}

}  // namespace pfc
