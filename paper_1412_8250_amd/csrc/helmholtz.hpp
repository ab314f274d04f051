// Shared declarations of the shifted-system (Helmholtz) solvers: the system
// table, complex helpers and the batch context.  Two schedules exist:
//  * stepped (default): every COCG phase is one launch over the tiles of all
//    running systems, iterations are replayed from a captured HIP graph;
//  * persistent: one cooperative launch in which groups of workgroups run
//    whole solves, taking systems from a device queue.
#pragma once

#include <vector>

#include "multigrid.hpp"
#include "stencil_core.hpp"
#include "tuning.hpp"
#include "vec.hpp"

namespace ofdft {

// H_IDLE marks systems that do not take part in a pass.
enum HDone { H_RUNNING = 0, H_CONVERGED = 1, H_BREAKDOWN = 2, H_NONFINITE = 3, H_MAXIT = 4, H_IDLE = 5 };

// Slots of the stepped schedule's ring (see helmholtz_stepped.hip): 4 or 2.
constexpr int kRingMax = 4;
// A cycle that forms rho itself; one (a single level) that leaves it to the dot phase.
enum { kPrecondCycle = 1, kPrecondDots = 2 };

struct HSys {
    int nx, ny, nz;
    int nunits;
    int brick, pad;           // stepped stencil phases: 1 = bricks (bg), 0 = marched tiles (tg)
    TileGeom tg;
    BrickGeom bg;
    int64_t n;
    Coef<double> coef;
    Coef<float> coef32;
    double kre, kim;          // adjacent: the multigrid cycle reads them as {Re, Im}
    void *x, *r, *p, *Ap;
    // stepped schedule: the vectors the directions are built from (residuals, or
    // z = M r with a preconditioner) of the iterations whose p and x are still
    // to be brought up to date; iteration k's in slot k % ring.  Without a
    // preconditioner slot 0 is r.  The persistent schedule's second p is slot 1.
    void *q[kRingMax];
    int ring, precond;        // precond: 0, kPrecondCycle or kPrecondDots
    const void *f;
};

struct HState;
struct GroupCtl;

// Device state of a system in the stepped schedule.
struct StepState {
    double rr_re, rr_im;     // r^T r (preconditioned: r^T z) of the current residual
    double al[kRingMax][2];  // alpha and beta {re, im} of the iterations in the ring
    double be[kRingMax][2];  // (slot iter % ring)
    double pa[2];            // p^T A p of the last direction
    double rn2, fn2, tol2;   // |r|^2, |f|^2, tol^2 |f|^2
    int iter, done, maxit, pad;      // iter % ring directions are still to be applied to x
};

// rho = r^T z and |z|^2 of the preconditioned iteration and what follows from
// them: the first call of a solve (iter 0) sets rho, later ones
// beta = rho_new / rho and rho.  st: the first system of the launch.
struct StepRho {
    static constexpr int kSums = 3;
    static constexpr bool kExtra = false;
    using Extra = double2;
    StepState *st;
    int ring;
    __device__ void prepare() {}
    __device__ static void point(double (&acc)[3], double2 z, double2 r) {
        acc[0] += r.x * z.x - r.y * z.y;
        acc[1] += r.x * z.y + r.y * z.x;
        acc[2] += z.x * z.x + z.y * z.y;
    }
    __device__ void finish(int q, const double (&t)[3]) const {
        StepState *sj = st + q;
        if (!isfinite(t[0]) || !isfinite(t[1]) || !isfinite(t[2])) {
            sj->done = H_NONFINITE;
        } else if (t[0] * t[0] + t[1] * t[1] <= 1e-60 * sj->rn2 * t[2]) {
            sj->done = H_BREAKDOWN;
        } else {
            if (sj->iter > 0) {
                const double rr_re = sj->rr_re, rr_im = sj->rr_im;
                const double d2 = rr_re * rr_re + rr_im * rr_im;
                double *be = sj->be[sj->iter % ring];
                be[0] = (t[0] * rr_re + t[1] * rr_im) / d2;
                be[1] = (t[1] * rr_re - t[0] * rr_im) / d2;
            }
            sj->rr_re = t[0];
            sj->rr_im = t[1];
        }
    }
};

template <typename T> struct CX;
template <> struct CX<double2> {
    using S = double;
    __device__ static double2 mk(double a, double b) { return make_double2(a, b); }
};
template <> struct CX<float2> {
    using S = float;
    __device__ static float2 mk(double a, double b) { return make_float2((float)a, (float)b); }
};

template <typename T>
__device__ inline T cfma(T a, T b, T c) {     // a*b + c (complex)
    T o;
    o.x = c.x + a.x * b.x - a.y * b.y;
    o.y = c.y + a.x * b.y + a.y * b.x;
    return o;
}


template <typename T>
__device__ inline const Coef<typename VT<T>::S> &coef_of(const HSys &s);
template <>
__device__ inline const Coef<double> &coef_of<double2>(const HSys &s) { return s.coef; }
template <>
__device__ inline const Coef<float> &coef_of<float2>(const HSys &s) { return s.coef32; }

// Tile shape actually used for complex element type T: complex128 keeps
// the z queue in registers only with one or two rows per thread, so its
// 16-row shapes map to the 64 x 8 tile of 512 threads.
template <typename T>
inline int cocg_shape(int shape) {
    if (sizeof(T) == 16 && (shape == SHAPE_64x4x4 || shape == SHAPE_64x8x2)) return SHAPE_64x8x1;
    return shape;
}

template <typename T, class F>
inline int dispatch_cocg_shape(int shape, F &&f) {
    if constexpr (sizeof(T) == 16) {
        switch (cocg_shape<T>(shape)) {
            case SHAPE_32x8x2: return f(ShapeTag<32, 8, 2>{});
            case SHAPE_64x8x1: return f(ShapeTag<64, 8, 1>{});
            default: return f(ShapeTag<64, 4, 2>{});
        }
    } else {
        return dispatch_shape(shape, f);
    }
}

}  // namespace ofdft

namespace ofdft {
// Default z-chunk target of the stepped schedule (planes per chunk).
constexpr int kStepPlanes = 80;
}  // namespace ofdft

struct ofdft_batch {
    int nsys = 0, radius = 6;
    ofdft_dtype dtype = OFDFT_C128;
    std::vector<ofdft_grid> grids;
    std::vector<void *> allocs;
    // per system workspaces (complex128: r, p, ring slots 1 .. ring - 1, Ap; complex64 adds r128, f32, x32)
    std::vector<void *> r, p, Ap, r128, f32, x32;
    std::vector<void *> slot[ofdft::kRingMax];   // slot[0] unused
    int ring = 2;                                // 2 (compact) or 4: slots in use
    ofdft::HSys *d_sys = nullptr;
    ofdft::HState *d_st = nullptr;
    int *d_order = nullptr;
    ofdft::GroupCtl *d_ctl = nullptr;
    double (*d_part)[4] = nullptr;    // 2 * groups_cap rows of 4 partial sums
    unsigned int *d_queue = nullptr;
    int *d_abort = nullptr;
    double *d_totals = nullptr;   // 2 per system
    ofdft::RedBuf rb{};
    int groups_cap = 0;
    // launch configuration: shape (< 0: default), persistent group size
    // (0: stepped schedule) and the stepped schedule's z-chunk target (planes)
    int shape = -1, P = 0, zplanes = ofdft::kStepPlanes;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    // stepped schedule
    ofdft::StepState *d_step = nullptr, *h_step = nullptr;   // per system (host copy pinned)
    int *d_ublk = nullptr, *d_vblk = nullptr;                 // block prefix sums (nsys + 1)
    // marched systems, then systems on bricks; per XCD: prefix sums of its share of
    // every system's tiles (2 x 8 x (nsys + 1); none of the other class)
    int *d_xpre = nullptr;
    int step_grid[2] = {0, 0};   // stencil-phase workgroups of each class: 8 x the longest XCD share
    size_t step_lds = 0;         // LDS bytes of the brick launches
    unsigned int *d_ctr = nullptr;                           // per-system arrival counters
    double *d_spart = nullptr;                               // per-system partial slots
    int step_shape = -1, step_units = 0, step_vblocks = 0;
    std::vector<int> h_ublk, h_vblk, h_brick;
    hipGraphExec_t step_graph = nullptr;
    hipStream_t step_cap = nullptr;
    int step_graph_key[5] = {-1, -1, -1, -1, -1};
    // preconditioner (OFDFT_PRECOND_*): z = M r per system
    int precond = 0;
    double *d_kap = nullptr;      // {Re, Im} for ofdft_batch_apply_preconditioner
    std::vector<void *> z;        // ring slot 0 of the preconditioned iteration
    std::vector<ofdft::Multigrid *> mg_of, mg_own;
    // consecutive systems on one grid form a group: one hierarchy holds their
    // level arrays (system j is member mg_q[j]) and one launch per kernel runs
    // their cycles; groups as (first system, count)
    std::vector<int> mg_q;
    std::vector<std::pair<int, int>> mg_groups;
    void **d_rtab = nullptr, **d_ztab = nullptr;   // device tables: r[j]; ring slot k of system j at [k nsys + j]
    // the groups' cycles run on kMgLanes side streams (group g on lane
    // g % lanes), forked from and joined back into the solve's stream, so
    // the latency-bound coarse levels of different groups overlap
    std::vector<hipStream_t> mg_lane;
    std::vector<hipEvent_t> mg_join;
    hipEvent_t mg_fork = nullptr;
};

namespace ofdft {

constexpr int kMgLanes = 4;
constexpr int kMgGroupMax = 64;     // systems per grouped cycle

// Stepped schedule: run COCG on the systems in `which` (system table `hs`
// already uploaded; maxit[j] per system) to relative residual tol.  On return
// iters[j] and done[j] hold the per-system iteration counts and outcomes.
int stepped_run(ofdft_batch *b, bool c64, int shape, const std::vector<HSys> &hs,
                const std::vector<int> &which, const std::vector<int> &maxit, double tol,
                std::vector<int> &iters, std::vector<int> &done, hipStream_t s);
void stepped_free(ofdft_batch *b);
// z-chunk length of the stepped stencil phases on grid g for chunks of about
// `planes` planes (depends only on g, the shape and the batch's setting, so a
// system's reduction order does not depend on the rest of the batch).
int stepped_zlen(const ofdft_grid &g, bool c64, int shape, int planes = kStepPlanes);

}  // namespace ofdft
