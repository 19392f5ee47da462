// launch.hpp -- host-side launchers of the PFC kernels, one set per dtype (float, double).
// Each returns the HIP error of its launch; shapes are validated by the caller (pfc_api.cpp).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "types.hpp"

namespace pfc {

// Geometry of a 2D/3D grid as the kernels see it.
struct Geom {
    int ndim;
    int64_t n0, n1, nx;  // 2D: n0 = y, n1 = 1 (unused), nx = x; 3D: z, y, x
    int64_t M;           // nx / 2
    int64_t nrows;       // rows of the last-axis pass: n1 (3D) or 1 (2D)
    int64_t xrows;       // rows of the x pass: n0 * nrows
    int lt_shift;        // log2 of the twiddle table length
    bool nt;             // non-temporal loads/stores of the grids in the step and FFT passes
    // twiddle table of each pass, as an entry offset from the plan's twiddle buffer: 0 (the
    // power-of-two tables) or the own table of a length that is not a power of two
    int64_t tw_x, tw_y, tw_last;
    // layout of the packed spectra (Pack in types.hpp): row pitch (0: M), plane-block and column-chunk
    // shifts; zero is the plain layout
    int64_t Mp = 0;
    int zs = 0, cs = 0;
    int xnat = 0;  // x passes in natural row order
    bool init = false;  // forward transforms of the state set-up (InitXPlan, InitAxisPlan in FP32)
};

// The Pack of a geometry.
inline Pack pack_of(const Geom &g) { return Pack{g.nrows, g.Mp > 0 ? g.Mp : g.M, g.zs, g.cs, g.xnat}; }

// A layout the kernels can address: shifts in range, pitch >= M, and with plane blocks a pitch of
// whole column chunks and a last-axis length of whole blocks.  Every launcher of a packed-layout
// kernel checks it, so a bad geometry is an error, not an out-of-bounds access.
inline bool layout_ok(const Geom &g)
{
    const int64_t Mp = g.Mp > 0 ? g.Mp : g.M;
    if (g.zs < 0 || g.zs > 3 || g.cs < 0 || g.cs > 4 || Mp < g.M) return false;
    if (g.zs == 0) return true;
    return g.ndim == 3 && Mp % (int64_t(1) << g.cs) == 0 && g.n0 % (int64_t(1) << g.zs) == 0;
}

// Lengths other than powers of two that have compiled schedules (factors 2, 3, 5, 7); a grid axis
// of length n needs n here (y and last axis) or n / 2 here (x).
constexpr int kMixedLengths[] = {6, 10, 12, 14, 15, 20, 30, 60, 150, 375, 700, 750, 1400};
inline bool mixed_length(int64_t n)
{
    for (int m : kMixedLengths)
        if (n == m) return true;
    return false;
}

// `variant`: candidate schedule of the pass (0 = default); only the step's passes (x r2c with the
// cube, y forward/inverse, last-axis STEP, x c2r) have more than one candidate.
template <typename T>
hipError_t launch_x_r2c(const Geom &g, const T *in, cx<T> *out, bool cube, const cx<T> *tw, hipStream_t s,
                        int variant = 0);

template <typename T>
hipError_t launch_x_c2r(const Geom &g, const cx<T> *in, T *out, const cx<T> *tw, hipStream_t s, int variant = 0);

// fused x pass between two steps, in place on the packed spectrum: x c2r (1/N; also stored to `real`
// unless that is null), cube, x r2c; on the default x schedules, where x_fused_ok says the geometry has it
template <typename T>
hipError_t launch_x_c2r_r2c(const Geom &g, cx<T> *data, T *real, const cx<T> *tw, hipStream_t s);
// the same between two adjoint steps: lambda_n as launch_x_c2r_adjoint, not stored, then its x r2c into data
template <typename T>
hipError_t launch_x_adj_r2c(const Geom &g, cx<T> *data, const cx<T> *nu, const T *psi_n, const T *psi_np1, T c3,
                            double *partial, int64_t slots, bool add, int64_t *nblocks, const cx<T> *tw, hipStream_t s);
template <typename T>
bool x_fused_ok(const Geom &g);
// whether the last-axis passes can address blocks of 2^zs z planes (their element steps are
// multiples of the block)
template <typename T>
bool z_blocks_ok(const Geom &g, int zs);

// adjoint epilogue: out = mu - c3 psi_n^2 nu; partial[block] = (add: +=) sum nu psi_np1.  Returns the
// number of partials through *nblocks; nothing is launched if they are more than `slots`.
template <typename T>
hipError_t launch_x_c2r_adjoint(const Geom &g, const cx<T> *mu, const cx<T> *nu, const T *psi_n, const T *psi_np1,
                                T *out, T c3, double *partial, int64_t slots, bool add, int64_t *nblocks, const cx<T> *tw,
                                hipStream_t s);
// rows per workgroup, at least, of the adjoint epilogue's pass in 3D
constexpr int kAdjRows3 = 4;

// y-axis (3D middle axis) complex FFT, in place; dir = -1 forward, +1 inverse.
template <typename T>
hipError_t launch_y_c2c(const Geom &g, cx<T> *data, int dir, const cx<T> *tw, hipStream_t s, int variant = 0);

// last-axis complex FFT, forward, out of place, packed in and out (no update).
template <typename T>
hipError_t launch_last_fwd(const Geom &g, const cx<T> *src, cx<T> *dst, const cx<T> *tw, hipStream_t s);

// last-axis complex FFT (dir = -1 forward, +1 inverse), out of place or in place, packed in and out.
template <typename T>
hipError_t launch_last_c2c(const Geom &g, const cx<T> *src, cx<T> *dst, int dir, const cx<T> *tw, hipStream_t s);

// Hydrodynamic passes (hydro.hpp).
// Last-axis pass of an operation: HYDRO_DERIV o0 = inv(s), o1 = inv(i k_last s); HYDRO_MU the same of
// mu = nl fwd(a) + (r + L) s; HYDRO_PSI updates s with fwd(a) = FFT(psi^3) and fwd(b) = FFT(v . grad psi),
// o0 = inv(s); HYDRO_VEL updates s with fwd(a) = FFT(psi grad_j mu), o0 = inv(s).  o0 may be a or b.
enum HydroOp { HYDRO_DERIV = 0, HYDRO_MU = 1, HYDRO_PSI = 2, HYDRO_VEL = 3 };
template <typename T>
hipError_t launch_hydro_last(const Geom &g, int op, const cx<T> *a, const cx<T> *b, cx<T> *s, cx<T> *o0, cx<T> *o1,
                             const HydroArgs &h, const cx<T> *tw, hipStream_t s_);
// 3D middle axis, inverse: dk = inv(i k_y data), then data = inv(data) in place
template <typename T>
hipError_t launch_hydro_y(const Geom &g, cx<T> *data, cx<T> *dk, double fk, const cx<T> *tw, hipStream_t s);
// x pass: field_j = x c2r of spec[j] (for the last component, x, of i k_x spec[j]); with `out`, out = x
// r2c of sum_j w[j] field_j (may be a spec); without, spec[j] = x r2c of w[0] field_j
template <typename T>
struct HydroFlow {
    cx<T> *spec[3];
    const T *w[3];
    cx<T> *out;
    double fkx;
};
template <typename T>
hipError_t launch_hydro_x(const Geom &g, const HydroFlow<T> &f, const cx<T> *tw, hipStream_t s);
// x pass of the new density: real = x c2r of in, out = x r2c of real^3 (out may be in)
template <typename T>
hipError_t launch_hydro_psi_x(const Geom &g, const cx<T> *in, T *real, cx<T> *out, const cx<T> *tw, hipStream_t s);

enum LastMode { LAST_STEP = 0, LAST_R2C_NATURAL = 1, LAST_C2R_NATURAL = 2, LAST_ADJOINT = 3 };

template <typename T>
hipError_t launch_last(const Geom &g, int mode, const cx<T> *src, cx<T> *dst, cx<T> *dst2, cx<T> *state,
                       const ModelParams<T> &mp, const cx<T> *tw, hipStream_t s, int variant = 0);

// number of candidate schedules of each step pass for this geometry (index as pfc_step_timed's
// passes); used by the autotuner
int step_candidates(const Geom &g, int pass);

// reductions; every launcher uses exactly kReduceBlocks partials
constexpr int kReduceBlocks = 1024;
template <typename T>
hipError_t launch_set_mass(const T *psi, int64_t n, double *partial, cx<T> *state, hipStream_t s);
template <typename T>
hipError_t launch_energy(const Geom &g, const T *psi, const cx<T> *state, const double fk[3], double r, double q1sq,
                         double R1, int model, double dV, double *partial, double *out, hipStream_t s);
template <typename T>
hipError_t launch_export(const Geom &g, const cx<T> *state, cx<T> *out, hipStream_t s);
hipError_t launch_accumulate(const double *partial, int np, double coef, double *acc, hipStream_t s);

// Batched form: a group of `count` instances of one shape and one choice of schedules, at table[first].
struct BatchGroup {
    int n0, M, vx, vy, vc, first, count;
};
// Small groups share their launches, those on the default schedules by class of y lengths, those on tuned ones
// all together: the unit of a group, 0 where it has launches of its own.
template <typename T>
int batch_unit(const BatchGroup &g);
// groups of a launch: a class has at most 4 y lengths with 6 of x
constexpr int kBatchUnitGroups = 24;
enum { BATCH_X_FWD = 0, BATCH_X_INV = 1, BATCH_X_FUSED = 2 };  // x r2c with the cube, x c2r, both between steps
// one pass of the unit g[0 .. ng)
template <typename T>
hipError_t launch_batch_x(const BatchGroup *g, int ng, int pass, const BatchInst<T> *table, const cx<T> *tw, int lt_shift,
                          hipStream_t s);
// y forward, update, y inverse
template <typename T>
hipError_t launch_batch_y(const BatchGroup *g, int ng, const BatchInst<T> *table, const cx<T> *tw, int lt_shift,
                          hipStream_t s);
// workgroups of a group's y pass
template <typename T>
int64_t batch_y_workgroups(const BatchGroup &g);
constexpr int kBatchMaxInstHost = 256;
// number of candidates of batched pass `pass` (0 x forward, 1 y, 2 x inverse) for an n0 x 2M instance
int batch_candidates(int n0, int M, int pass);

}  // namespace pfc
