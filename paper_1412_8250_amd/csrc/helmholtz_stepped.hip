// Stepped schedule of the batched COCG solver for the shifted systems
// (-L_h + kappa_j) u_j = f_j (Section 3.1; COCG = conjugate gradients with
// the unconjugated bilinear form x^T y, valid because -L_h + kappa is complex
// symmetric).
//
// Each COCG phase is ONE launch over all running systems of the batch:
//  * stencil phase: the stencil runs on r alone (A r = -L r + kappa r); the
//    image of the new direction p = r + beta p_old follows point by point from
//    the previous one, Ap = A r + beta Ap_old (A is linear), so only one array
//    is read with a halo, and p itself isn't needed: p^T A p = r^T A p +
//    beta p_old^T A p, where p_old^T A p = Ap_old^T r + beta p_old^T Ap_old is
//    zero but for rounding (with a single-precision cycle as preconditioner
//    that isn't small: left out, the solutions moved 5 times further).  The
//    two products r^T A p and Ap_old^T r are reduced.  The grid holds
//    the stencil tiles of every system, so eight 320^3 systems give
//    thousands of workgroups per launch.  Each XCD takes one contiguous
//    eighth of every system's tiles (neighbouring tiles share their halos
//    in that XCD's L2, and the systems still running keep every XCD busy
//    when the others have converged);
//  * vector phase: r -= alpha Ap into the next slot of a ring of residuals,
//    r^T r and |r|^2 reduced.  Every ring-th vector phase (ring = 4; 2 in
//    compact batches) brings p and x up to date from the
//    ring and the kept alphas and betas: p = r_k + beta_k p, x += alpha_k p.
// Per iteration that moves 6 vectors and (ring + 3) / ring for p and x: 7.75
// in place of the 10 that the update of p and x in each iteration takes
// (6 cells of 24 to 96 points an axis, 8 shifts each, to 1e-10: 66 -> 63 ms).
// The scalars of every system (alpha, beta, r^T r, status) live on the
// device: the last workgroup of a system to finish a phase combines that
// system's partial sums (fixed order, so results do not depend on timing or
// on the other systems of the batch) and updates its scalars.  Converged
// systems' workgroups exit at once.  Iterations are captured once in a HIP
// graph and replayed; the host only polls the status array between replays.
// No workgroup ever waits for another inside a launch.
//
// With a preconditioner M (one multigrid cycle per system, complex
// symmetric) the iteration is preconditioned COCG: after the vector phase
// z = M r is formed by the cycle's own launches, the last of which also
// reduces rho = r^T z and sets beta = rho_new / rho, and the stencil phase runs
// on z:
// p = z + beta p_old, Ap = A z + beta Ap_old, and so for p^T A p.  The ring
// then holds z; r is updated in place.
#include <algorithm>
#include <cmath>

#include "helmholtz.hpp"

namespace ofdft {

namespace {

constexpr int kStepIters = 4;          // iterations per captured graph
static_assert(kStepIters % kRingMax == 0 && kStepIters % 2 == 0, "a captured block ends at its first ring slot");
constexpr int kVecThreadsStep = 256;
constexpr int kVecMaxBlocks = 1024;    // per system

// System of logical block b: start[j] <= b < start[j + 1].
__device__ inline int find_sys(const int *start, int nsys, int b) {
    int lo = 0, hi = nsys;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (start[mid] <= b) lo = mid;
        else hi = mid;
    }
    return lo;
}

template <typename T>
struct StepLoadX {
    GPtr<T> x;
    __device__ T operator()(int64_t i) const { return x[i]; }
};


template <typename T>
struct StepEpiInit {     // r = f - (-L x + kappa x); acc {r^T r re, im, |r|^2, |f|^2}
    GPtr<T> f, r;
    T kappa;
    double acc[4];
    T fv[4];
    __device__ void pre(int q, int64_t i) { fv[q] = f[i]; }
    __device__ void point(int q, int64_t i, T c, T s) {
        const T ax = cfma(kappa, c, T{-s.x, -s.y});
        const T fi = fv[q];
        const T rv{fi.x - ax.x, fi.y - ax.y};
        r.st(i, rv);
        const double a = rv.x, b = rv.y;
        acc[0] += a * a - b * b;
        acc[1] += 2.0 * a * b;
        acc[2] += a * a + b * b;
        acc[3] += (double)fi.x * fi.x + (double)fi.y * fi.y;
    }
};

// Centre = r (z when preconditioned), s = L r.  Ap = (-L r + kappa r) +
// beta Ap_old, updated in place (each point is read and written by the same
// thread).  acc {r^T Ap re, im, r^T Ap_old re, im}.  The first iteration (beta = 0, no previous
// image) reads no Ap_old and is a kernel of its own: with a run-time flag the
// loads and their use sit in branches, and the compiler then waits for the
// halo fetches of the previous plane before it reuses their registers.
template <typename T, bool First>
struct StepEpiPAp {
    GPtr<T> Ap;
    T kappa, beta;
    double acc[4];
    T ao[4];
    __device__ void pre(int q, int64_t i) {
        if constexpr (!First) ao[q] = Ap[i];
    }
    __device__ void point(int q, int64_t i, T c, T s) {
        T a = cfma(kappa, c, T{-s.x, -s.y});
        if constexpr (!First) {
            a = cfma(beta, ao[q], a);
            acc[2] += (double)c.x * ao[q].x - (double)c.y * ao[q].y;
            acc[3] += (double)c.x * ao[q].y + (double)c.y * ao[q].x;
        }
        Ap.st(i, a);
        acc[0] += (double)c.x * a.x - (double)c.y * a.y;
        acc[1] += (double)c.x * a.y + (double)c.y * a.x;
    }
};

enum StepPhase { PH_INIT = 0, PH_PAP = 1, PH_PAP_FIRST = 2 };

// A system's tile by the march or, for small grids, by the brick kernel.
template <typename T, int TX, int TYT, int RY>
struct StepMarch {
    static constexpr int kThreads = TX * TYT;
    template <class Load, class Epi>
    __device__ static void run(const HSys &h, const Load &ld, Epi &ep, int unit) {
        __shared__ T lds[StencilLds<T, TX, TYT, RY>::kElems];
        stencil_tile<T, TX, TYT, RY>(h.tg, coef_of<T>(h), ld, ep, unit, lds);
    }
};
template <typename T>
struct StepBrick {
    static constexpr int kThreads = kBrickThreads;
    template <class Load, class Epi>
    __device__ static void run(const HSys &h, const Load &ld, Epi &ep, int unit) {
        extern __shared__ __align__(16) unsigned char brick_lds[];
        stencil_brick<T, 4>(h.bg, coef_of<T>(h), ld, ep, unit, reinterpret_cast<T *>(brick_lds));
    }
};

// Stencil phases.  part: 4 slots per unit, system j's region starts at
// 4 * ublk[j] and is laid out [k][unit].
template <typename T, class Tile, int Phase>
__global__ void __launch_bounds__(Tile::kThreads)
step_stencil(const HSys *sys, StepState *st, const int *ublk, const int *xpre, int nsys,
             unsigned int *ctr, double *part, double tol, int slot) {
    using CT = CX<T>;
    __shared__ double scratch[4 * (Tile::kThreads / 64)];
    // workgroup b runs on XCD b % 8; that XCD's list holds, system after
    // system, the tiles [n x / 8, n (x + 1) / 8) of each system of n tiles
    constexpr int kXcd = 8;
    const int x = blockIdx.x % kXcd, l = blockIdx.x / kXcd;
    const int *xp = xpre + x * (nsys + 1);
    if (l >= xp[nsys]) return;
    const int j = find_sys(xp, nsys, l);
    StepState *sj = st + j;
    const int done = sj->done;
    if (done != H_RUNNING) return;
    const HSys &h = sys[j];
    const int nunits = ublk[j + 1] - ublk[j];
    const int unit = (int)(((int64_t)nunits * x) / kXcd) + (l - xp[j]);
    double *pj = part + 4 * (size_t)ublk[j];
    const T kappa = CT::mk(h.kre, h.kim);
    if constexpr (Phase == PH_INIT) {
        StepLoadX<T> ld{GPtr<T>(h.x)};
        StepEpiInit<T> ep{GPtr<T>(h.f), GPtr<T>(h.r), kappa, {0, 0, 0, 0}, {}};
        Tile::run(h, ld, ep, unit);
        double acc[4] = {ep.acc[0], ep.acc[1], ep.acc[2], ep.acc[3]};
        block_sum<4>(acc, scratch);
        double t[4];
        if (reduce_grid<4>(acc, pj, nunits, unit, ctr + (size_t)j * kArriveWords, scratch, t)) {
            sj->rr_re = t[0];
            sj->rr_im = t[1];
            sj->rn2 = t[2];
            sj->fn2 = t[3];
            sj->tol2 = tol * tol * t[3];
            sj->iter = 0;
            int d = !isfinite(t[2]) ? H_NONFINITE : (t[2] <= sj->tol2 ? H_CONVERGED : H_RUNNING);
            if (d == H_RUNNING && sj->maxit <= 0) d = H_MAXIT;
            sj->done = d;
        }
    } else {
        // PH_PAP_FIRST runs iteration 0 of every running system, PH_PAP the
        // later ones (the host launches the first right after the init phase)
        StepLoadX<T> ld{GPtr<T>(h.q[slot])};
        StepEpiPAp<T, Phase == PH_PAP_FIRST> ep{GPtr<T>(h.Ap), kappa, CT::mk(sj->be[slot][0], sj->be[slot][1]),
                                                {0, 0, 0, 0}, {}};
        Tile::run(h, ld, ep, unit);
        constexpr int kSums = Phase == PH_PAP_FIRST ? 2 : 4;
        double acc[kSums];
        for (int k = 0; k < kSums; ++k) acc[k] = ep.acc[k];
        block_sum<kSums>(acc, scratch);
        double t[kSums];
        if (reduce_grid<kSums>(acc, pj, nunits, unit, ctr + (size_t)j * kArriveWords, scratch, t)) {
            if constexpr (kSums == 4) {         // + beta (Ap_old^T r + beta p_old^T Ap_old)
                const double be_re = sj->be[slot][0], be_im = sj->be[slot][1];
                const double u = t[2] + (be_re * sj->pa[0] - be_im * sj->pa[1]);
                const double v = t[3] + (be_re * sj->pa[1] + be_im * sj->pa[0]);
                t[0] += be_re * u - be_im * v;
                t[1] += be_re * v + be_im * u;
            }
            sj->pa[0] = t[0];
            sj->pa[1] = t[1];
            const double den = t[0] * t[0] + t[1] * t[1];
            if (!isfinite(den)) {
                sj->done = H_NONFINITE;
            } else if (den == 0.0) {
                sj->done = H_BREAKDOWN;
            } else {
                sj->al[slot][0] = (sj->rr_re * t[0] + sj->rr_im * t[1]) / den;
                sj->al[slot][1] = (sj->rr_im * t[0] - sj->rr_re * t[1]) / den;
            }
        }
    }
}

// p and x of one point brought up to date by the ring's first `cnt` directions.
template <typename T>
__device__ inline void ring_point(const T (&q)[kRingMax], int cnt, const T *al, const T *be, T &p, T &x) {
#pragma unroll
    for (int k = 0; k < kRingMax; ++k)
        if (k < cnt) {
            p = cfma(be[k], p, q[k]);
            x = cfma(al[k], p, x);
        }
}

// Vector phase of the iteration in ring slot `slot`: r -= alpha Ap (into the
// next slot; in place when preconditioned), with Ring > 0 (the last slot of a
// ring of Ring) also p and x; then beta (unpreconditioned) and status.  part
// region of system j starts at 4 * vblk[j] (the caller offsets part past the
// stencil slots).
template <typename T, int Ring>
__global__ void __launch_bounds__(kVecThreadsStep)
step_update(const HSys *sys, StepState *st, const int *vblk, int nsys, unsigned int *ctr,
            double *part, int slot) {
    using CT = CX<T>;
    __shared__ double scratch[3 * (kVecThreadsStep / 64)];
    const int b = blockIdx.x;
    const int j = find_sys(vblk, nsys, b);
    StepState *sj = st + j;
    if (sj->done != H_RUNNING) return;
    const HSys &h = sys[j];
    const int lb = b - vblk[j], nb = vblk[j + 1] - vblk[j];
    const bool pre = h.precond != 0;            // rho and beta come from the dot phase
    const int next = Ring ? 0 : slot + 1;
    const GPtr<T> r(pre ? h.r : h.q[slot]), rn(pre ? h.r : h.q[next]), Ap(h.Ap);
    const T nal = CT::mk(-sj->al[slot][0], -sj->al[slot][1]);
    double acc[3] = {0.0, 0.0, 0.0};
    const int64_t stride = (int64_t)nb * kVecThreadsStep;
    auto residual = [&](int64_t i, T rv) {
        rn.st(i, rv);
        const double a = rv.x, c = rv.y;
        acc[0] += a * a - c * c;
        acc[1] += 2.0 * a * c;
        acc[2] += a * a + c * c;
    };
    if constexpr (Ring > 0) {
        const GPtr<T> x(h.x), p(h.p);
        T al[kRingMax], be[kRingMax];
        GPtr<T> q[kRingMax];
        for (int k = 0; k < Ring; ++k) {
            al[k] = CT::mk(sj->al[k][0], sj->al[k][1]);
            be[k] = CT::mk(sj->be[k][0], sj->be[k][1]);
            q[k] = GPtr<T>(h.q[k]);
        }
        const bool have = sj->iter >= Ring;     // p holds a direction
        for (int64_t i = (int64_t)lb * kVecThreadsStep + threadIdx.x; i < h.n; i += stride) {
            T qv[kRingMax];
            for (int k = 0; k < Ring; ++k) qv[k] = q[k][i];
            const T rv = pre ? r[i] : qv[Ring - 1];
            T pv{0, 0}, xv = x[i];
            if (have) pv = p[i];
            residual(i, cfma(nal, Ap[i], rv));
            ring_point<T>(qv, Ring, al, be, pv, xv);
            p.st(i, pv);
            x.st(i, xv);
        }
    } else {
        for (int64_t i = (int64_t)lb * kVecThreadsStep + threadIdx.x; i < h.n; i += stride)
            residual(i, cfma(nal, Ap[i], r[i]));
    }
    block_sum<3>(acc, scratch);
    double t[3];
    if (reduce_grid<3>(acc, part + 4 * (size_t)vblk[j], nb, lb, ctr + (size_t)j * kArriveWords, scratch, t)) {
        if (!pre) {
            const double rr_re = sj->rr_re, rr_im = sj->rr_im;
            const double d2 = rr_re * rr_re + rr_im * rr_im;
            sj->be[next][0] = (t[0] * rr_re + t[1] * rr_im) / d2;
            sj->be[next][1] = (t[1] * rr_re - t[0] * rr_im) / d2;
            sj->rr_re = t[0];
            sj->rr_im = t[1];
        }
        sj->rn2 = t[2];
        const int iter = sj->iter + 1;
        sj->iter = iter;
        int d = H_RUNNING;
        if (!isfinite(t[2])) d = H_NONFINITE;
        else if (t[2] <= sj->tol2) d = H_CONVERGED;
        else if (!pre && t[0] * t[0] + t[1] * t[1] <= 1e-60 * t[2] * t[2]) d = H_BREAKDOWN;
        else if (iter >= sj->maxit) d = H_MAXIT;
        sj->done = d;
    }
}

// x of every system that stopped between two updates of x: the directions in
// the ring, iter % ring of them.
template <typename T>
__global__ void __launch_bounds__(kVecThreadsStep)
step_finish(const HSys *sys, const StepState *st, const int *vblk, int nsys) {
    using CT = CX<T>;
    const int b = blockIdx.x;
    const int j = find_sys(vblk, nsys, b);
    const StepState *sj = st + j;
    const HSys &h = sys[j];
    const int cnt = sj->iter % h.ring;
    if (!cnt) return;
    const int lb = b - vblk[j], nb = vblk[j + 1] - vblk[j];
    const GPtr<T> x(h.x), p(h.p);
    T al[kRingMax], be[kRingMax];
    GPtr<T> q[kRingMax];
#pragma unroll
    for (int k = 0; k < kRingMax; ++k) {
        al[k] = CT::mk(sj->al[k][0], sj->al[k][1]);
        be[k] = CT::mk(sj->be[k][0], sj->be[k][1]);
        q[k] = GPtr<T>(h.q[k < cnt ? k : 0]);
    }
    const bool have = sj->iter >= h.ring;
    const int64_t stride = (int64_t)nb * kVecThreadsStep;
    for (int64_t i = (int64_t)lb * kVecThreadsStep + threadIdx.x; i < h.n; i += stride) {
        T qv[kRingMax];
#pragma unroll
        for (int k = 0; k < kRingMax; ++k)
            if (k < cnt) qv[k] = q[k][i];
        T pv{0, 0}, xv = x[i];
        if (have) pv = p[i];
        ring_point<T>(qv, cnt, al, be, pv, xv);
        x.st(i, xv);
    }
}

// Dot phase of the preconditioned iteration for systems whose grid is itself
// the coarsest one (longer cycles form rho in their last kernel).
__global__ void __launch_bounds__(kVecThreadsStep)
step_dot(const HSys *sys, StepState *st, const int *vblk, int nsys, unsigned int *ctr, double *part) {
    __shared__ double scratch[3 * (kVecThreadsStep / 64)];
    const int b = blockIdx.x;
    const int j = find_sys(vblk, nsys, b);
    StepState *sj = st + j;
    const HSys &h = sys[j];
    if (sj->done != H_RUNNING || h.precond != kPrecondDots) return;
    const int lb = b - vblk[j], nb = vblk[j + 1] - vblk[j];
    const GPtr<double2> r(h.r), z(h.q[sj->iter % h.ring]);
    double acc[3] = {0.0, 0.0, 0.0};
    const int64_t stride = (int64_t)nb * kVecThreadsStep;
    for (int64_t i = (int64_t)lb * kVecThreadsStep + threadIdx.x; i < h.n; i += stride) {
        StepRho::point(acc, z[i], r[i]);
    }
    block_sum<3>(acc, scratch);
    double t[3];
    if (reduce_grid<3>(acc, part + 4 * (size_t)vblk[j], nb, lb, ctr + (size_t)j * kArriveWords, scratch, t))
        StepRho{st, h.ring}.finish(j, t);
}

template <typename T, class Tile>
int launch_phase(ofdft_batch *b, int cls, int phase, dim3 threads, size_t lds, double tol, int slot, hipStream_t s) {
    auto kern = phase == PH_INIT ? step_stencil<T, Tile, PH_INIT>
                : phase == PH_PAP_FIRST ? step_stencil<T, Tile, PH_PAP_FIRST>
                : step_stencil<T, Tile, PH_PAP>;
    hipLaunchKernelGGL(kern, dim3(b->step_grid[cls]), threads, lds, s, b->d_sys, b->d_step, b->d_ublk,
                       b->d_xpre + cls * 8 * (b->nsys + 1), b->nsys, b->d_ctr, b->d_spart, tol, slot);
    OFDFT_CHECK_HIP(hipGetLastError());
    return OFDFT_OK;
}

// One launch per class of systems present (marched tiles, bricks).
template <typename T>
int launch_stencil_phase(ofdft_batch *b, int shape, int phase, double tol, int slot, hipStream_t s) {
    if (b->step_grid[0])
        OFDFT_TRY(dispatch_cocg_shape<T>(shape, [&](auto sh) {
            using S = decltype(sh);
            return launch_phase<T, StepMarch<T, S::TX, S::TYT, S::RY>>(b, 0, phase, dim3(S::TX, S::TYT), 0, tol, slot,
                                                                       s);
        }));
    if (b->step_grid[1])
        OFDFT_TRY((launch_phase<T, StepBrick<T>>(b, 1, phase, dim3(kBrickThreads), b->step_lds, tol, slot, s)));
    return OFDFT_OK;
}

template <typename T>
int launch_update(ofdft_batch *b, int slot, hipStream_t s) {
    auto kern = slot < b->ring - 1 ? step_update<T, 0> : b->ring == 2 ? step_update<T, 2> : step_update<T, kRingMax>;
    hipLaunchKernelGGL(kern, dim3(b->step_vblocks), dim3(kVecThreadsStep), 0, s, b->d_sys,
                       b->d_step, b->d_vblk, b->nsys, b->d_ctr, b->d_spart + 4 * (size_t)b->step_units, slot);
    OFDFT_CHECK_HIP(hipGetLastError());
    return OFDFT_OK;
}

// Whether a system of the batch needs the dot phase.
bool dot_phase(const ofdft_batch *b) {
    return std::any_of(b->mg_own.begin(), b->mg_own.end(), [](const Multigrid *mg) { return !mg_forms_dots(*mg); });
}

// z = M r (into ring slot `slot`) of every preconditioned system, then rho = r^T z (and beta).
// Systems that are not running skip both inside the kernels.  The cycles run
// on the batch's side streams (forked from s and joined back; inside a graph
// capture this makes parallel branches).  Timed: the host reads the
// statuses first and launches (and times) only the cycles of running
// systems, one after another on s, so each cycle's duration is its own;
// otherwise the caller accounts them.
int precondition(ofdft_batch *b, int slot, hipStream_t s, bool timed) {
    if (timed) {
        OFDFT_CHECK_HIP(hipMemcpyAsync(b->h_step, b->d_step, sizeof(StepState) * b->nsys, hipMemcpyDeviceToHost, s));
        OFDFT_CHECK_HIP(hipStreamSynchronize(s));
    }
    static_assert(sizeof(HSys) % sizeof(double) == 0 && sizeof(StepState) % sizeof(int) == 0,
                  "per-system shift and status strides");
    const int lanes = timed ? 0 : (int)b->mg_lane.size();
    if (lanes) OFDFT_CHECK_HIP(hipEventRecord(b->mg_fork, s));
    for (int k = 0; k < lanes; ++k) OFDFT_CHECK_HIP(hipStreamWaitEvent(b->mg_lane[k], b->mg_fork, 0));
    if (timed) {
        // one cycle per running system, one after another on s, each timed
        for (int j = 0; j < b->nsys; ++j) {
            if (b->h_step[j].done != H_RUNNING) continue;
            // bytes are added after the pass from the iteration counts
            ProfScope ps(K_MULTIGRID_C, 0.0, s);
            OFDFT_TRY(mg_apply_shifted(*b->mg_of[j], b->mg_q[j], (const double2 *)b->r[j],
                                       (double2 *)(slot ? b->slot[slot][j] : b->z[j]), StepRho{b->d_step + j, b->ring}, &b->d_sys[j].kre, &b->d_step[j].done, s));
        }
    } else {
        // one grouped cycle per group: shift {kre, kim} and status of system j
        // at d_sys[j] and d_step[j]; converged systems' workgroups return at once
        for (size_t g = 0; g < b->mg_groups.size(); ++g) {
            const int j0 = b->mg_groups[g].first, cnt = b->mg_groups[g].second;
            hipStream_t q = lanes ? b->mg_lane[g % lanes] : s;
            OFDFT_TRY(mg_apply_shifted_group(*b->mg_of[j0], cnt, (const double2 *const *)(b->d_rtab + j0),
                                             (double2 *const *)(b->d_ztab + (size_t)slot * b->nsys + j0),
                                             StepRho{b->d_step + j0, b->ring}, &b->d_sys[j0].kre,
                                             (int)(sizeof(HSys) / sizeof(double)), &b->d_step[j0].done,
                                             (int)(sizeof(StepState) / sizeof(int)), q));
        }
    }
    for (int k = 0; k < lanes; ++k) {
        OFDFT_CHECK_HIP(hipEventRecord(b->mg_join[k], b->mg_lane[k]));
        OFDFT_CHECK_HIP(hipStreamWaitEvent(s, b->mg_join[k], 0));
    }
    if (!dot_phase(b)) return OFDFT_OK;
    ProfScope ps(K_COCG_UPDATE, 0.0, s, timed);
    hipLaunchKernelGGL(step_dot, dim3(b->step_vblocks), dim3(kVecThreadsStep), 0, s, b->d_sys,
                       b->d_step, b->d_vblk, b->nsys, b->d_ctr, b->d_spart + 4 * (size_t)b->step_units);
    OFDFT_CHECK_HIP(hipGetLastError());
    return OFDFT_OK;
}

// `iters` iterations of all phases after the first one (ring slots 1, 2, ..;
// a multiple of the ring).  Timed: each launch is accounted and
// timed on its own; otherwise (graph capture) the caller accounts replays.
template <typename T>
int step_iterations(ofdft_batch *b, int shape, int iters, hipStream_t s, bool timed) {
    for (int k = 0; k < iters; ++k) {
        const int slot = (k + 1) % b->ring;
        {
            ProfScope ps(K_COCG, 0.0, s, timed);
            OFDFT_TRY(launch_stencil_phase<T>(b, shape, PH_PAP, 0.0, slot, s));
        }
        {
            ProfScope ps(K_COCG_UPDATE, 0.0, s, timed);
            OFDFT_TRY(launch_update<T>(b, slot, s));
        }
        if (b->precond) OFDFT_TRY(precondition(b, (slot + 1) % b->ring, s, timed));
    }
    return OFDFT_OK;
}

// Iteration 0 of every running system (eager: the captured block holds
// later iterations only).  Accounted like the init phase.
template <typename T>
int first_iteration(ofdft_batch *b, int shape, hipStream_t s, bool timed) {
    {
        ProfScope ps(K_COCG, 0.0, s);
        OFDFT_TRY(launch_stencil_phase<T>(b, shape, PH_PAP_FIRST, 0.0, 0, s));
    }
    {
        ProfScope ps(K_COCG_UPDATE, 0.0, s);
        OFDFT_TRY(launch_update<T>(b, 0, s));
    }
    if (b->precond) {
        OFDFT_TRY(precondition(b, 1, s, timed));
        if (!timed) {
            if (dot_phase(b)) prof_add(K_COCG_UPDATE, 0.0, 1);
            prof_add(K_MULTIGRID_C, 0.0, b->nsys);
        }
    }
    return OFDFT_OK;
}

template <typename T>
int graph_get(ofdft_batch *b, int shape) {
    const int key[5] = {shape, (int)sizeof(T), b->step_units, b->precond, b->step_grid[1]};
    if (b->step_graph && std::equal(key, key + 5, b->step_graph_key)) return OFDFT_OK;
    if (b->step_graph) {
        (void)hipGraphExecDestroy(b->step_graph);
        b->step_graph = nullptr;
    }
    if (!b->step_cap) OFDFT_CHECK_HIP(hipStreamCreateWithFlags(&b->step_cap, hipStreamNonBlocking));
    hipGraph_t graph = nullptr;
    OFDFT_CHECK_HIP(hipStreamBeginCapture(b->step_cap, hipStreamCaptureModeThreadLocal));
    const int rc = step_iterations<T>(b, shape, kStepIters, b->step_cap, false);
    const hipError_t e = hipStreamEndCapture(b->step_cap, &graph);
    if (rc != OFDFT_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return rc;
    }
    OFDFT_CHECK_HIP(e);
    const hipError_t ei = hipGraphInstantiate(&b->step_graph, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    OFDFT_CHECK_HIP(ei);
    for (int i = 0; i < 5; ++i) b->step_graph_key[i] = key[i];
    return OFDFT_OK;
}

// Block tables of the current system table (units from the uploaded tile
// geometries, vector blocks from the sizes) and the partial-slot buffer.
int prepare_layout(ofdft_batch *b, const std::vector<HSys> &hs, size_t elem, hipStream_t s) {
    const int nsys = b->nsys;
    std::vector<int> ublk(nsys + 1, 0), vblk(nsys + 1, 0), brick(nsys, 0);
    size_t lds = 0;
    for (int j = 0; j < nsys; ++j) {
        brick[j] = hs[j].brick;
        if (brick[j]) lds = std::max(lds, brick_lds_bytes(hs[j].bg, 4, elem));
        ublk[j + 1] = ublk[j] + hs[j].nunits;
        const int64_t want = (hs[j].n + 8 * kVecThreadsStep - 1) / (8 * kVecThreadsStep);
        vblk[j + 1] = vblk[j] + (int)std::max<int64_t>(1, std::min<int64_t>(want, kVecMaxBlocks));
    }
    b->step_lds = lds;
    if (ublk == b->h_ublk && vblk == b->h_vblk && brick == b->h_brick) return OFDFT_OK;
    if (b->step_graph) {                    // captured with the old tables
        OFDFT_CHECK_HIP(hipStreamSynchronize(s));
        (void)hipGraphExecDestroy(b->step_graph);
        b->step_graph = nullptr;
    }
    // per-XCD shares of every system's tiles (see step_stencil), class by class
    std::vector<int> xpre(2 * 8 * (size_t)(nsys + 1), 0);
    for (int cls = 0; cls < 2; ++cls) {
        int longest = 0;
        for (int x = 0; x < 8; ++x) {
            int *xp = xpre.data() + (cls * 8 + x) * (nsys + 1);
            for (int j = 0; j < nsys; ++j) {
                const int64_t nu = brick[j] == cls ? ublk[j + 1] - ublk[j] : 0;
                xp[j + 1] = xp[j] + (int)(nu * (x + 1) / 8 - nu * x / 8);
            }
            longest = std::max(longest, xp[nsys]);
        }
        b->step_grid[cls] = 8 * longest;
    }
    if (!b->d_ublk) {
        OFDFT_CHECK_HIP(hipMalloc(&b->d_xpre, sizeof(int) * 16 * (nsys + 1)));
        OFDFT_CHECK_HIP(hipMalloc(&b->d_ublk, sizeof(int) * (nsys + 1)));
        OFDFT_CHECK_HIP(hipMalloc(&b->d_vblk, sizeof(int) * (nsys + 1)));
        OFDFT_CHECK_HIP(hipMalloc(&b->d_ctr, sizeof(unsigned int) * kArriveWords * nsys));
        OFDFT_CHECK_HIP(hipMalloc(&b->d_step, sizeof(StepState) * nsys));
        OFDFT_CHECK_HIP(hipHostMalloc(&b->h_step, sizeof(StepState) * nsys, hipHostMallocDefault));
        OFDFT_CHECK_HIP(hipMemsetAsync(b->d_ctr, 0, sizeof(unsigned int) * kArriveWords * nsys, s));
    }
    const size_t slots = 4 * ((size_t)ublk[nsys] + (size_t)vblk[nsys]);
    const size_t have = 4 * ((size_t)(b->h_ublk.empty() ? 0 : b->h_ublk[nsys]) +
                             (size_t)(b->h_vblk.empty() ? 0 : b->h_vblk[nsys]));
    if (!b->d_spart || slots > have) {
        if (b->d_spart) OFDFT_CHECK_HIP(hipFree(b->d_spart));
        b->d_spart = nullptr;
        OFDFT_CHECK_HIP(hipMalloc(&b->d_spart, sizeof(double) * slots));
    }
    OFDFT_CHECK_HIP(hipMemcpyAsync(b->d_ublk, ublk.data(), sizeof(int) * (nsys + 1), hipMemcpyHostToDevice, s));
    OFDFT_CHECK_HIP(hipMemcpyAsync(b->d_xpre, xpre.data(), sizeof(int) * xpre.size(), hipMemcpyHostToDevice, s));
    OFDFT_CHECK_HIP(hipMemcpyAsync(b->d_vblk, vblk.data(), sizeof(int) * (nsys + 1), hipMemcpyHostToDevice, s));
    OFDFT_CHECK_HIP(hipStreamSynchronize(s));
    b->h_ublk = ublk;
    b->h_vblk = vblk;
    b->h_brick = brick;
    b->step_units = ublk[nsys];
    b->step_vblocks = vblk[nsys];
    return OFDFT_OK;
}

template <typename T>
int run_t(ofdft_batch *b, int shape, const std::vector<HSys> &hs, const std::vector<int> &which, const std::vector<int> &maxit,
          double tol, std::vector<int> &iters, std::vector<int> &done, hipStream_t s) {
    const int nsys = b->nsys;
    for (int j = 0; j < nsys; ++j) {
        b->h_step[j] = StepState{};
        b->h_step[j].done = H_IDLE;
        b->h_step[j].maxit = maxit[j];
    }
    for (int j : which) b->h_step[j].done = H_RUNNING;
    OFDFT_CHECK_HIP(hipMemcpyAsync(b->d_step, b->h_step, sizeof(StepState) * nsys, hipMemcpyHostToDevice, s));
    const bool timed = prof_timed(K_COCG) || prof_timed(K_COCG_UPDATE) ||
                       (b->precond && prof_timed(K_MULTIGRID_C));
    {
        ProfScope ps(K_COCG, 0.0, s);
        OFDFT_TRY(launch_stencil_phase<T>(b, shape, PH_INIT, tol, 0, s));
    }
    if (b->precond) {
        OFDFT_TRY(precondition(b, 0, s, timed));
        if (!timed) {
            if (dot_phase(b)) prof_add(K_COCG_UPDATE, 0.0, 1);
            prof_add(K_MULTIGRID_C, 0.0, nsys);
        }
    }
    int reps = 1;
    std::vector<double> rn2_0(nsys, 0.0);     // residual after the init phase
    bool first = true;
    for (;;) {
        OFDFT_CHECK_HIP(hipMemcpyAsync(b->h_step, b->d_step, sizeof(StepState) * nsys, hipMemcpyDeviceToHost, s));
        OFDFT_CHECK_HIP(hipStreamSynchronize(s));
        bool running = false;
        for (int j : which) running = running || b->h_step[j].done == H_RUNNING;
        if (!running) break;
        if (first) {
            for (int j : which) rn2_0[j] = b->h_step[j].rn2;
            first = false;
            OFDFT_TRY(first_iteration<T>(b, shape, s, timed));
        } else {
            // replays until the slowest running system is predicted to converge,
            // from its mean residual reduction per iteration so far
            double need = 0.0;
            bool known = true;
            for (int j : which) {
                const StepState &q = b->h_step[j];
                if (q.done != H_RUNNING) continue;
                const double rate = q.iter > 0 && rn2_0[j] > 0 ? std::log(q.rn2 / rn2_0[j]) / q.iter : 0.0;
                if (!(rate < -1e-3) || !std::isfinite(rate)) {
                    known = false;
                    break;
                }
                need = std::max(need, std::log(q.tol2 / q.rn2) / rate);
            }
            reps = known ? (int)std::ceil(std::max(need, 1.0) / kStepIters) : reps * 2;
            reps = std::max(1, std::min(reps, 32));
        }
        if (timed) {
            OFDFT_TRY(step_iterations<T>(b, shape, reps * kStepIters, s, true));
        } else {
            OFDFT_TRY(graph_get<T>(b, shape));
            for (int k = 0; k < reps; ++k) OFDFT_CHECK_HIP(hipGraphLaunch(b->step_graph, s));
            prof_add(K_COCG, 0.0, reps * kStepIters);
            prof_add(K_COCG_UPDATE, 0.0, reps * kStepIters * (b->precond && dot_phase(b) ? 2 : 1));
            if (b->precond) prof_add(K_MULTIGRID_C, 0.0, (int64_t)reps * kStepIters * nsys);
        }
    }
    // the directions still in the ring (read them, x and p; write x)
    double fin = 0.0;
    for (int j : which)
        if (const int cnt = b->h_step[j].iter % b->ring)
            fin += (cnt + (b->h_step[j].iter >= b->ring ? 3.0 : 2.0)) * sizeof(T) * (double)hs[j].n;
    if (fin > 0.0) {
        ProfScope ps(K_COCG_UPDATE, fin, s);
        hipLaunchKernelGGL(step_finish<T>, dim3(b->step_vblocks), dim3(kVecThreadsStep), 0, s, b->d_sys, b->d_step,
                           b->d_vblk, b->nsys);
        OFDFT_CHECK_HIP(hipGetLastError());
    }
    for (int j = 0; j < nsys; ++j) {
        iters[j] = b->h_step[j].iter;
        done[j] = b->h_step[j].done;
    }
    return OFDFT_OK;
}

}  // namespace

// Chunks of about `planes` planes (default 80): long enough for little
// queue warm-up, short enough that one or two systems still running (the
// tail of a batch) spread over more workgroups than the chip's CUs
// (measured: 80 beat 160 and 40 at 320^3; the autotuner times others); they
// shrink down to 8 planes while a system would have fewer than 32 tiles.
int stepped_zlen(const ofdft_grid &g, bool, int shape, int planes) {
    int tx, ty;
    shape_extent(shape, tx, ty);
    const int64_t tiles = (int64_t)((g.nx + tx - 1) / tx) * ((g.ny + ty - 1) / ty);
    planes = std::max(planes, 8);
    int chunks = std::max(1, (g.nz + planes - 1) / planes);
    while (tiles * chunks < 32 && g.nz / (chunks + 1) >= 8) ++chunks;
    return (g.nz + chunks - 1) / chunks;
}

int stepped_run(ofdft_batch *b, bool c64, int shape, const std::vector<HSys> &hs,
                const std::vector<int> &which, const std::vector<int> &maxit, double tol,
                std::vector<int> &iters, std::vector<int> &done, hipStream_t s) {
    if (b->precond && c64) return OFDFT_INVALID_ARG;
    OFDFT_TRY(prepare_layout(b, hs, c64 ? sizeof(float2) : sizeof(double2), s));
    if (c64) return run_t<float2>(b, shape, hs, which, maxit, tol, iters, done, s);
    return run_t<double2>(b, shape, hs, which, maxit, tol, iters, done, s);
}

void stepped_free(ofdft_batch *b) {
    if (b->step_graph) (void)hipGraphExecDestroy(b->step_graph);
    if (b->step_cap) (void)hipStreamDestroy(b->step_cap);
    if (b->d_xpre) (void)hipFree(b->d_xpre);
    if (b->d_ublk) (void)hipFree(b->d_ublk);
    if (b->d_vblk) (void)hipFree(b->d_vblk);
    if (b->d_ctr) (void)hipFree(b->d_ctr);
    if (b->d_step) (void)hipFree(b->d_step);
    if (b->h_step) (void)hipHostFree(b->h_step);
    if (b->d_spart) (void)hipFree(b->d_spart);
    b->step_graph = nullptr;
    b->step_cap = nullptr;
    b->d_ublk = b->d_vblk = b->d_xpre = nullptr;
    b->d_ctr = nullptr;
    b->d_step = b->h_step = nullptr;
    b->d_spart = nullptr;
}

}  // namespace ofdft
