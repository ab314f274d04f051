// Geometric multigrid V-cycle (see multigrid.hpp) and the Poisson form that
// uses it as the preconditioner of CG.
#include <algorithm>
#include <cmath>
#include <utility>

#include "fcg.hpp"
#include "helmholtz.hpp"
#include "multigrid.hpp"
#include "profile.hpp"

namespace ofdft {

namespace {

constexpr int kMgCoarseThreads = 1024;

struct MgDims {
    int nx, ny, nz;
    double cx, cy, cz, diag;
    double kre, kim;          // shift kappa of A = -Delta_h + kappa
    int64_t n;
};

MgDims dims_of(const MgLevel &L, double2 kappa) {
    return MgDims{L.nx, L.ny, L.nz, L.cx, L.cy, L.cz, 2.0 * (L.cx + L.cy + L.cz), kappa.x, kappa.y, L.n};
}

// Element types: the cycle's input f and output z are FP64 (real or complex);
// the levels' arrays are stored, and their arithmetic done, in S (FP64 or
// FP32, real or complex).  R is S's real type, C the complex scalar of that
// precision (the Jacobi factor and the shift).
template <typename S> struct MgT;
template <> struct MgT<double> { using R = double; using C = double2; };
template <> struct MgT<float> { using R = float; using C = float2; };
template <> struct MgT<double2> { using R = double; using C = double2; };
template <> struct MgT<float2> { using R = float; using C = float2; };

template <typename To> __device__ inline To cv(double v);
template <typename To> __device__ inline To cv(float v);
template <typename To> __device__ inline To cv(double2 v);
template <typename To> __device__ inline To cv(float2 v);
template <> __device__ inline double cv<double>(double v) { return v; }
template <> __device__ inline float cv<float>(double v) { return (float)v; }
template <> __device__ inline double cv<double>(float v) { return (double)v; }
template <> __device__ inline float cv<float>(float v) { return v; }
template <> __device__ inline double2 cv<double2>(double2 v) { return v; }
template <> __device__ inline float2 cv<float2>(double2 v) { return make_float2((float)v.x, (float)v.y); }
template <> __device__ inline double2 cv<double2>(float2 v) { return make_double2(v.x, v.y); }
template <> __device__ inline float2 cv<float2>(float2 v) { return v; }

__device__ inline double mg_scale(double2 s, double v) { return s.x * v; }
__device__ inline float mg_scale(float2 s, float v) { return s.x * v; }
__device__ inline double2 mg_scale(double2 s, double2 v) {
    return make_double2(s.x * v.x - s.y * v.y, s.x * v.y + s.y * v.x);
}
__device__ inline float2 mg_scale(float2 s, float2 v) {
    return make_float2(s.x * v.x - s.y * v.y, s.x * v.y + s.y * v.x);
}
__device__ inline double mg_axpy(double a, double x, double y) { return ::fma(a, x, y); }
__device__ inline float mg_axpy(float a, float x, float y) { return fmaf(a, x, y); }
__device__ inline double2 mg_axpy(double a, double2 x, double2 y) {
    return make_double2(::fma(a, x.x, y.x), ::fma(a, x.y, y.y));
}
__device__ inline float2 mg_axpy(float a, float2 x, float2 y) {
    return make_float2(fmaf(a, x.x, y.x), fmaf(a, x.y, y.y));
}

template <typename C> __device__ inline C mk_c(double a, double b);
template <> __device__ inline double2 mk_c<double2>(double a, double b) { return make_double2(a, b); }
template <> __device__ inline float2 mk_c<float2>(double a, double b) { return make_float2((float)a, (float)b); }

// Per-launch shift source: when `kap` is given, kappa is read from device
// memory (so a captured launch follows the current shift); when `run` is
// given the kernel returns at once unless *run == 0 (a converged system of a
// batch).  System q of a launch reads kap + q kstride and run + q rstride.
struct MgShift {
    const double *kap;
    const int *run;
    int kstride, rstride;
    __device__ bool skip(int q) const { return run && run[(int64_t)q * rstride] != 0; }
};

// An array of every system of a launch: system q's part starts at
// base + q stride, or at tab[q] (a device table of the callers' arrays).
template <typename P>
struct MgArr {
    P *base;
    int64_t stride;
    P *const *tab;
    __device__ P *at(int q) const { return tab ? tab[q] : (base ? base + (int64_t)q * stride : nullptr); }
};

// Returns false when system q is to be skipped; otherwise sets d's shift.
__device__ inline bool take_shift(const MgShift &sh, MgDims &d, int q) {
    if (sh.skip(q)) return false;
    if (sh.kap) {
        d.kre = sh.kap[(int64_t)q * sh.kstride];
        d.kim = sh.kap[(int64_t)q * sh.kstride + 1];
    }
    return true;
}

// omega / (diag + kappa)
template <typename C>
__device__ inline C jacobi_factor(const MgDims &d, double w) {
    const double re = d.diag + d.kre, im = d.kim, den = re * re + im * im;
    return mk_c<C>(w * re / den, -w * im / den);
}

// Columns of a workgroup: thread t takes columns t, t + NT, ... (SL of them)
// of the tile's (W + 2 HALO) x (H + 2 HALO) region less `trim` on its far
// sides, and walks them down z together, one plane per step.  `off` is the
// column's periodic (x, y) offset in a plane; `depth` its distance from the
// region's near/far edge (a stage of stencil reach k is formed where depth
// >= k); own marks the tile's own points inside the grid.
template <int SL>
struct MgCols {
    int off[SL], depth[SL];
    bool own[SL];
};

template <int NT, int SL>
__device__ __forceinline__ void mg_cols(const MgDims &d, const MgTile &tl, int x0, int y0, int halo, int RW,
                                        int RH, MgCols<SL> &c) {
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const int k = threadIdx.x + i * NT;
        const int ly = k / RW, lx = k - ly * RW;
        const bool act = ly < RH;
        int gx = (x0 - halo + lx) % d.nx, gy = (y0 - halo + ly) % d.ny;
        gx += gx < 0 ? d.nx : 0;
        gy += gy < 0 ? d.ny : 0;
        c.off[i] = act ? gy * d.nx + gx : 0;
        c.depth[i] = act ? min(min(lx, RW - 1 - lx), min(ly, RH - 1 - ly)) : -1;
        c.own[i] = act && lx >= halo && lx < halo + tl.W && ly >= halo && ly < halo + tl.H &&
                   x0 + lx - halo < d.nx && y0 + ly - halo < d.ny;
    }
}

// A c for the periodic 7-point operator A = -Delta_h + kappa from the centre c
// and its neighbours' values, in the cycle's fixed order of operations.
template <typename S, typename C>
__device__ __forceinline__ S mg_op(const MgDims &d, C kap, S c, S xp, S xm, S yp, S ym, S zm, S zp) {
    using V = VT<S>;
    using R = typename MgT<S>::R;
    S a = V::mul((R)d.diag, c);
    a = mg_axpy((R)-d.cx, V::add(xp, xm), a);
    a = mg_axpy((R)-d.cy, V::add(yp, ym), a);
    a = mg_axpy((R)-d.cz, V::add(zm, zp), a);
    return V::add(a, mg_scale(kap, c));
}

// Tile of the workgroup: origin, planes [z0, z0 + zl) and system.
struct MgWhere {
    int x0, y0, z0, zl, q, b;      // b: the workgroup's number in its system
};
__device__ inline MgWhere mg_where(const MgTile &tl, int nz) {
    int b = xcd_remap(blockIdx.x, gridDim.x);
    MgWhere m;
    m.b = b % (tl.tx * tl.ty * tl.tz);
    m.x0 = (b % tl.tx) * tl.W;
    b /= tl.tx;
    m.y0 = (b % tl.ty) * tl.H;
    b /= tl.ty;
    m.z0 = (b % tl.tz) * tl.zl;
    m.q = b / tl.tz;
    m.zl = min(tl.zl, nz - m.z0);
    return m;
}

// Products formed by the upward half of level 0: kSums sums of point(z, r,
// extra) per system, handed to finish(system, sums) by the last workgroup.
struct MgNoDot {
    static constexpr int kSums = 0;
    static constexpr bool kExtra = false;
    using Extra = double;
};
template <class Dot>
struct MgDot {
    Dot dot;
    double *part;              // Multigrid::kDotSums cap slots per system
    unsigned int *ctr;         // kArriveWords per system
    int cap;
};

// State of the preconditioned CG below, on the device.
constexpr int kPcgRing = 4;
struct PDev {
    double *x;
    double rz, pAp, zAp, r2, tol2;
    double a[kPcgRing], b[kPcgRing];     // of the iterations in the ring
    int iters, maxit, done;
    int n_ap, n_step, n_dots;
};

struct PcgRho {          // {<z, Ap>, <r, z>}: beta and the next rho
    static constexpr int kSums = 2;
    static constexpr bool kExtra = true;
    using Extra = double;
    const double *Ap;
    PDev *D;
    int slot, next;
    __device__ void prepare() {}
    __device__ double extra(int64_t i) const { return GPtr<double>(Ap)[i]; }
    __device__ static void point(double (&acc)[2], double z, double r, double ap) {
        acc[0] = ::fma(z, ap, acc[0]);
        acc[1] = ::fma(r, z, acc[1]);
    }
    __device__ void finish(int, const double (&t)[2]) const {
        const double b = -D->a[slot] * t[0] / D->rz;
        D->b[next] = isfinite(b) ? b : 0.0;
        D->zAp = t[0];
        D->rz = t[1];
        D->n_dots += 1;
    }
};

// Downward half of a level, one pass over f: the two pre-smoothing sweeps from
// u = 0 (with the Jacobi factor s = omega / (diag + kappa), u1 = s f and
// u2 = u1 + s (f - A u1) = s (2 f - s A f)), the residual r = f - A u2 and its
// full weighting fc[I] = sum over the 27 fine points around 2I of
// (1/8) w(dx) w(dy) w(dz) r, w(0) = 1, w(+-1) = 1/2 (= P^T / 8).  Stores u2 and
// fc; r is never stored.
//
// Bound by HBM: 12.5 B/point for FP64 f and FP32 levels (read f; write u and 1/8
// fc) where three separate passes moved 32.5.  The tile is
// marched along z with one plane of f, u and r each in LDS (double-buffered:
// every step writes one buffer and reads the one the step before wrote, so
// one barrier per plane serves all three stages, each one plane behind the
// one that feeds it); the z neighbours stay in registers; f is fetched two
// planes ahead.  The (x, y) halo of 3 (2 on the far side) and 5 warm-up planes
// per z chunk are re-read through L2.  Measured, the cycle (back to back,
// FP64 vectors and FP32 levels, five passes per level before): 320^3 723 ->
// 393 us, 160^3 169 -> 102 us, 96^3 109 -> 58 us; complex 160^3 260 -> 157 us.
template <typename TF, typename S, int NT, int SL>
__global__ void __launch_bounds__(NT) mg_down(MgDims d, MgDims cd, MgTile tl, double w, MgArr<const TF> fa,
                                              MgArr<S> ua, MgArr<S> cfa, MgShift sh) {
    using V = VT<S>;
    using R = typename MgT<S>::R;
    using C = typename MgT<S>::C;
    __shared__ S fb[2][NT * SL], ub[2][NT * SL], rb[2][NT * SL];
    const MgWhere m = mg_where(tl, d.nz);
    if (!take_shift(sh, d, m.q)) return;
    // global-space views: a pointer from a table is generic to the compiler,
    // and flat loads would share the LDS wait counter
    const GPtr<TF> f(fa.at(m.q));
    const GPtr<S> u(ua.at(m.q)), fc(cfa.at(m.q));
    const int RW = tl.W + 5, RH = tl.H + 5;
    MgCols<SL> co;
    mg_cols<NT, SL>(d, tl, m.x0, m.y0, 3, RW, RH, co);
    const C s = jacobi_factor<C>(d, w), kap = mk_c<C>(d.kre, d.kim);
    const int64_t nxy = (int64_t)d.nx * d.ny;
    // the thread's coarse point of the tile: fine (2X, 2Y) is region column cc
    const int tid = threadIdx.x, cw = tl.W / 2;
    const int ciy = tid / cw, cix = tid - ciy * cw;
    const int X = m.x0 / 2 + cix, Y = m.y0 / 2 + ciy;
    const bool cown = ciy < tl.H / 2 && X < cd.nx && Y < cd.ny;
    const int cc = cown ? (3 + 2 * ciy) * RW + 3 + 2 * cix : RW + 1;
    const int64_t cxy = (int64_t)cd.nx * cd.ny;
    const int64_t crow = (int64_t)Y * cd.nx + X;

    TF fn[2][SL];                                  // f two planes ahead
    S f0[SL], f1[SL], u0[SL], u1[SL];              // f[p-2], f[p-1], u[p-3], u[p-2] of step plane p
    S q0 = V::zero(), q1 = V::zero();              // plane sums of the coarse point
    int kf = (m.z0 - 3) % d.nz;                    // plane of the next fetch
    kf += kf < 0 ? d.nz : 0;
    int p = kf;                                    // plane of the step (periodic)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int i = 0; i < SL; ++i) fn[j][i] = f[kf * nxy + co.off[i]];
        kf = kf + 1 == d.nz ? 0 : kf + 1;
    }
#pragma unroll
    for (int i = 0; i < SL; ++i) f0[i] = f1[i] = u0[i] = u1[i] = V::zero();

    // step t: f[p] enters (p = z0 - 3 + t), u[p-1], r[p-2] are formed, r[p-3] restricted
    auto step = [&](int t, auto pc) __attribute__((always_inline)) {
        constexpr int B = decltype(pc)::value, Q = B ^ 1;
        const bool live = t <= m.zl + 4;           // the last step only restricts
        if (live) {
            S f2[SL], un[SL];
#pragma unroll
            for (int i = 0; i < SL; ++i) f2[i] = cv<S>(fn[B][i]);
            if (t + 2 <= m.zl + 4) {
#pragma unroll
                for (int i = 0; i < SL; ++i) fn[B][i] = f[kf * nxy + co.off[i]];
                kf = kf + 1 == d.nz ? 0 : kf + 1;
            }
#pragma unroll
            for (int i = 0; i < SL; ++i) {
                const int c = tid + i * NT;
                fb[B][c] = f2[i];
                un[i] = V::zero();
                if (t >= 2 && co.depth[i] >= 1) {
                    const S af = mg_op<S>(d, kap, f1[i], fb[Q][c + 1], fb[Q][c - 1], fb[Q][c + RW], fb[Q][c - RW],
                                          f0[i], f2[i]);
                    un[i] = mg_scale(s, V::sub(V::add(f1[i], f1[i]), mg_scale(s, af)));
                    ub[B][c] = un[i];
                    if (co.own[i] && t >= 4 && t <= m.zl + 3)
                        u.st((p == 0 ? d.nz - 1 : p - 1) * nxy + co.off[i], un[i]);
                }
                if (t >= 4 && co.depth[i] >= 2) {
                    const S au = mg_op<S>(d, kap, u1[i], ub[Q][c + 1], ub[Q][c - 1], ub[Q][c + RW], ub[Q][c - RW],
                                          u0[i], un[i]);
                    rb[B][c] = V::sub(f0[i], au);
                }
                f0[i] = f1[i];
                f1[i] = f2[i];
                u0[i] = u1[i];
                u1[i] = un[i];
            }
            p = p + 1 == d.nz ? 0 : p + 1;
        }
        if (t >= 5 && cown) {
            S acc = V::zero();
#pragma unroll
            for (int b = -1; b <= 1; ++b) {
                const S *row = rb[Q] + cc + b * RW;
                const S rowsum = V::add(mg_axpy((R)0.5, V::add(row[-1], row[1]), V::zero()), row[0]);
                acc = mg_axpy(b == 0 ? (R)1 : (R)0.5, rowsum, acc);
            }
            if constexpr (B == 1) {                // odd fine plane: closes coarse plane Z, opens Z + 1
                if (t >= 7) {
                    const S sz = V::add(mg_axpy((R)0.5, V::add(q0, acc), V::zero()), q1);
                    fc.st(((m.z0 + t - 7) >> 1) * cxy + crow, V::mul((R)0.125, sz));
                }
                q0 = acc;
            } else {
                q1 = acc;
            }
        }
        __syncthreads();
    };
    for (int t = 0; t <= m.zl + 5; t += 2) {       // zl is even
        step(t, std::integral_constant<int, 0>{});
        step(t + 1, std::integral_constant<int, 1>{});
    }
}

// Upward half of a level: v = u + P uc (trilinear: per axis, fine index i takes
// coarse i/2 when i is even and the mean of coarse (i-1)/2 and (i+1)/2 when
// odd), then the two post-smoothing sweeps t = v + s (f - A v) and
// z = t + s (f - A t); v and t are never stored.
//
// Bound by HBM: 20.5 B/point for FP32 levels and FP64 f and z (read f, u, 1/8 uc;
// write z) where two passes moved 28.5 (with f in FP32).  The march of mg_down with halo 2 and
// four warm-up planes per z chunk: v[p], t[p-1] and z[p-2] are formed in the
// step of plane p.  A column keeps the (x, y)-interpolated coarse value of the
// two coarse planes around it; the next one's corners are fetched a step
// ahead.
//
// With a Dot (level 0 inside a Krylov loop) the products of z with r = f (and
// with A p) that the loop takes next are reduced here, from the z at hand and
// r re-read through the caches.  f is the caller's FP64 array also with FP32
// levels: a copy in FP32 would save here what the downward half would write.
// Bytes per point of FP64 vectors with FP32 levels, cycle and products, where a pass of
// its own read r and z: 49 -> 33 (with A p 57 -> 41).  Measured, whole solves:
// Poisson 96^3 1.61 -> 1.52 ms, 320^3 15.2 -> 14.1 (15.1 with the real
// operands loaded where they are used); eight shifted systems of 96^3 6.7 -> 6.4;
// an SCF step of 320^3 226 -> 212.
template <typename TF, typename S, typename TO, int NT, int SL, class Dot>
__global__ void __launch_bounds__(NT) mg_up(MgDims d, MgDims cd, MgTile tl, double w, MgArr<const TF> fa,
                                            MgArr<const S> ua, MgArr<const S> uca, MgArr<TO> za, MgShift sh,
                                            MgDot<Dot> dot) {
    using V = VT<S>;
    using R = typename MgT<S>::R;
    using C = typename MgT<S>::C;
    __shared__ S vb[2][NT * SL], tb[2][NT * SL];
    const MgWhere m = mg_where(tl, d.nz);
    if (!take_shift(sh, d, m.q)) return;
    const GPtr<TF> f(fa.at(m.q));
    const GPtr<S> u(ua.at(m.q)), uc(uca.at(m.q));
    const GPtr<TO> z(za.at(m.q));
    const int tid = threadIdx.x, RW = tl.W + 4, RH = tl.H + 4;
    MgCols<SL> co;
    mg_cols<NT, SL>(d, tl, m.x0, m.y0, 2, RW, RH, co);
    const C s = jacobi_factor<C>(d, w), kap = mk_c<C>(d.kre, d.kim);
    const int64_t nxy = (int64_t)d.nx * d.ny, cxy = (int64_t)cd.nx * cd.ny;
    // coarse corners of each column: (ya, xa), (ya, xb), (yb, xa), (yb, xb)
    int c00[SL], dxc[SL], dyc[SL];
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const int gy = co.off[i] / d.nx, gx = co.off[i] - gy * d.nx;
        const int xa = gx >> 1, ya = gy >> 1;
        const int xb = gx & 1 ? (xa + 1 == cd.nx ? 0 : xa + 1) : xa;
        const int yb = gy & 1 ? (ya + 1 == cd.ny ? 0 : ya + 1) : ya;
        c00[i] = ya * cd.nx + xa;
        dxc[i] = xb - xa;
        dyc[i] = (yb - ya) * cd.nx;
    }
    int p = (m.z0 - 2) % d.nz;                     // plane of the step (periodic)
    p += p < 0 ? d.nz : 0;
    int kf = p;                                    // plane of the next fetch
    S un[2][SL];
    TF fn[2][SL];
    S cn[4][SL];                                   // corners of the next coarse plane
    S ca[SL];                                      // corner sum on coarse plane floor(p / 2)
    auto corners = [&](int Z) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            const int64_t b = Z * cxy + c00[i];
            cn[0][i] = uc[b];
            cn[1][i] = uc[b + dxc[i]];
            cn[2][i] = uc[b + dyc[i]];
            cn[3][i] = uc[b + dyc[i] + dxc[i]];
        }
    };
    corners(p >> 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            un[j][i] = u[kf * nxy + co.off[i]];
            fn[j][i] = f[kf * nxy + co.off[i]];
        }
        kf = kf + 1 == d.nz ? 0 : kf + 1;
    }
    S f0[SL], f1[SL], v0[SL], v1[SL], t0[SL], t1[SL];   // f, v at p-2, p-1; t at p-3, p-2
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        ca[i] = V::add(V::add(cn[0][i], cn[1][i]), V::add(cn[2][i], cn[3][i]));
        f0[i] = f1[i] = v0[i] = v1[i] = t0[i] = t1[i] = V::zero();
    }
    [[maybe_unused]] double acc[Dot::kSums ? Dot::kSums : 1] = {};
    // the products' operands, a step ahead where that spills nothing (not
    // complex ones): issued before the step's fetches, so that waiting for them
    // leaves those in flight
    constexpr bool kAhead = Dot::kSums > 0 && sizeof(TO) == 8 && (sizeof(S) == 4 || SL < 4);
    [[maybe_unused]] TO dr[SL] = {};
    [[maybe_unused]] typename Dot::Extra de[SL] = {};
    if constexpr (Dot::kSums > 0) dot.dot.prepare();
    auto step = [&](int t, auto pc) __attribute__((always_inline)) {
        constexpr int B = decltype(pc)::value, Q = B ^ 1;
        S f2[SL], v2[SL];
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            f2[i] = cv<S>(fn[B][i]);
            S corr;
            if constexpr (B == 0) {                // even plane
                corr = V::mul((R)0.25, ca[i]);
            } else {
                const S cb = V::add(V::add(cn[0][i], cn[1][i]), V::add(cn[2][i], cn[3][i]));
                corr = mg_axpy((R)0.125, V::add(ca[i], cb), V::zero());
                ca[i] = cb;
            }
            v2[i] = V::add(un[B][i], corr);
        }
        const int64_t zo = (int64_t)(m.z0 + t - 4) * nxy;
        [[maybe_unused]] TO rv[SL];
        [[maybe_unused]] typename Dot::Extra ev[SL];
        if constexpr (kAhead) {
#pragma unroll
            for (int i = 0; i < SL; ++i) {
                rv[i] = dr[i];
                ev[i] = de[i];
                if (t >= 3 && t < m.zl + 3 && co.own[i]) {
                    dr[i] = f[zo + nxy + co.off[i]];
                    if constexpr (Dot::kExtra) de[i] = dot.dot.extra(zo + nxy + co.off[i]);
                }
            }
        }
        if constexpr (B == 0) corners((p >> 1) + 1 == cd.nz ? 0 : (p >> 1) + 1);
        if (t + 2 <= m.zl + 3) {
#pragma unroll
            for (int i = 0; i < SL; ++i) {
                un[B][i] = u[kf * nxy + co.off[i]];
                fn[B][i] = f[kf * nxy + co.off[i]];
            }
            kf = kf + 1 == d.nz ? 0 : kf + 1;
        }
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            const int c = tid + i * NT;
            vb[B][c] = v2[i];
            S tn = V::zero();
            if (t >= 2 && co.depth[i] >= 1) {
                const S av = mg_op<S>(d, kap, v1[i], vb[Q][c + 1], vb[Q][c - 1], vb[Q][c + RW], vb[Q][c - RW],
                                      v0[i], v2[i]);
                tn = V::add(v1[i], mg_scale(s, V::sub(f1[i], av)));
                tb[B][c] = tn;
            }
            if (t >= 4 && co.own[i]) {
                if constexpr (Dot::kSums > 0 && !kAhead) {
                    rv[i] = f[zo + co.off[i]];
                    if constexpr (Dot::kExtra) ev[i] = dot.dot.extra(zo + co.off[i]);
                }
                const S at = mg_op<S>(d, kap, t1[i], tb[Q][c + 1], tb[Q][c - 1], tb[Q][c + RW], tb[Q][c - RW],
                                      t0[i], tn);
                const TO zv = cv<TO>(V::add(t1[i], mg_scale(s, V::sub(f0[i], at))));
                z.st(zo + co.off[i], zv);
                if constexpr (Dot::kSums > 0) {
                    if constexpr (Dot::kExtra) Dot::point(acc, zv, rv[i], ev[i]);
                    else Dot::point(acc, zv, rv[i]);
                }
            }
            f0[i] = f1[i];
            f1[i] = f2[i];
            v0[i] = v1[i];
            v1[i] = v2[i];
            t0[i] = t1[i];
            t1[i] = tn;
        }
        p = p + 1 == d.nz ? 0 : p + 1;
        __syncthreads();
    };
    for (int t = 0; t <= m.zl + 3; t += 2) {       // zl is even
        step(t, std::integral_constant<int, 0>{});
        step(t + 1, std::integral_constant<int, 1>{});
    }
    if constexpr (Dot::kSums > 0) {
        constexpr int K = Dot::kSums;
        __shared__ double scratch[K * (NT / 64)];
        block_sum<K>(acc, scratch);
        double tot[K];
        if (reduce_grid<K>(acc, dot.part + (int64_t)m.q * Multigrid::kDotSums * dot.cap, tl.tx * tl.ty * tl.tz, m.b,
                           dot.ctr + (int64_t)m.q * kArriveWords, scratch, tot))
            dot.dot.finish(m.q, tot);
    }
}

// Exact solve on the coarsest grid (at most 16^3 points, one workgroup per
// system, FP64): A is diagonalised by the real Fourier basis (per axis the
// orthonormal cosines and sines of 2 pi k j / n, which share the eigenvalue
// 2 - 2 cos(2 pi k / n)), eigenvalue sum_a c_a (2 - 2 cos(2 pi k_a / n_a)) +
// kappa; with kappa = 0 the k = 0 (constant) component is set to zero.  The
// basis is real, so a complex system is two real ones up to the division.
//
// Bound by latency (six dependent axis passes in one workgroup).  An axis pass
// is the product of the basis matrix with all pencils of the axis, on the
// FP64 matrix cores: 16 pencils at a time, v_mfma_f64_16x16x4 over the axis
// (lane (n, kq) supplies Q[n][4 s + kq] and point 4 s + kq of pencil n in
// step s, and receives outputs kq + 4 i of pencil n), zero-padded to 16.  The
// lane's part of Q stays in registers for the pass.  The cycle's coarse solve
// at 10^3 / 12^3 took 18 / 30 us as a complex DFT with one LDS read per
// multiply, 11 / 13 us so (profiled, real).
constexpr int kMgTab = kMgCoarseMax * kMgCoarseMax;
typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ inline double2 mg_to_c(double v) { return make_double2(v, 0.0); }
__device__ inline double2 mg_to_c(float v) { return make_double2(v, 0.0); }
__device__ inline double2 mg_to_c(double2 v) { return v; }
__device__ inline double2 mg_to_c(float2 v) { return make_double2(v.x, v.y); }
__device__ inline void mg_from_c(double2 v, double &o) { o = v.x; }
__device__ inline void mg_from_c(double2 v, float &o) { o = (float)v.x; }
__device__ inline void mg_from_c(double2 v, double2 &o) { o = v; }
__device__ inline void mg_from_c(double2 v, float2 &o) { o = make_float2((float)v.x, (float)v.y); }

// tab: per axis the basis matrix Q (row k, column j, kMgCoarseMax apart), then
// per axis its transpose, then per axis 2 - 2 cos(2 pi k / n).
template <typename TI, typename TO>
__global__ void __launch_bounds__(kMgCoarseThreads) mg_coarse_solve(MgDims d, MgArr<const TI> fa, MgArr<TO> ua,
                                                                    MgShift sh, const double *__restrict__ tab) {
    constexpr int NC = VT<TI>::ncomp;
    constexpr int kRow = kMgCoarseMax + 1;         // odd row pitch: no bank conflicts along x
    constexpr int kPlane = kRow * kMgCoarseMax * kMgCoarseMax;
    __shared__ double a[NC * kPlane];
    constexpr int kTab = 6 * kMgTab + 3 * kMgCoarseMax;
    __shared__ double tl[kTab];
    const int q = blockIdx.x;                      // one workgroup per system
    if (!take_shift(sh, d, q)) return;
    const GPtr<TI> f(fa.at(q));
    const GPtr<TO> u(ua.at(q));
    const int nx = d.nx, ny = d.ny, nz = d.nz, n = (int)d.n;
    const int sy = nx | 1, sz = sy * ny;
    // i / m for the small ranges here (i < 2^13): exact, without the integer division
    auto quot = [](int i, float inv) { return (int)(((float)i + 0.5f) * inv); };
    const float inx = 1.0f / (float)nx, iny = 1.0f / (float)ny;
    const double *eig = tl + 6 * kMgTab;
#pragma unroll
    for (int j = 0; j < (kTab + kMgCoarseThreads - 1) / kMgCoarseThreads; ++j) {
        const int i = threadIdx.x + j * kMgCoarseThreads;
        if (i < kTab) tl[i] = tab[i];
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, pn = lane & 15, kq = lane >> 4;
    constexpr int kPer = kMgCoarseMax * kMgCoarseMax * kMgCoarseMax / kMgCoarseThreads;
    TI fv[kPer];                                   // every load in flight before the first use
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = threadIdx.x + j * kMgCoarseThreads;
        fv[j] = f[i < n ? i : 0];
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = threadIdx.x + j * kMgCoarseThreads;
        if (i < n) {
            const int r = quot(i, inx), o = r * sy + i - r * nx;
            const double2 v = mg_to_c(fv[j]);
            a[o] = v.x;
            if constexpr (NC == 2) a[kPlane + o] = v.y;
        }
    }
    __syncthreads();
    for (int pass = 0; pass < 6; ++pass) {         // Q on x, y, z, then Q^T on x, y, z
        const int ax = pass < 3 ? pass : pass - 3;
        const int len = ax == 0 ? nx : (ax == 1 ? ny : nz);
        const int stride = ax == 0 ? 1 : (ax == 1 ? sy : sz);
        const int m = ax == 0 ? ny : nx;           // pencils: (y, z), (x, z) or (x, y)
        const int sa = ax == 0 ? sy : 1, sb = ax == 2 ? sy : sz;
        const int pencils = n / len;
        double qv[4];                              // Q[pn][4 s + kq]; zero beyond the axis
#pragma unroll
        for (int st = 0; st < 4; ++st) qv[st] = tl[pass * kMgTab + pn * kMgCoarseMax + 4 * st + kq];
        for (int t0 = wave * 16; t0 < NC * pencils; t0 += (kMgCoarseThreads / 64) * 16) {
            const int t = min(t0 + pn, NC * pencils - 1);
            const int c = NC == 2 && t >= pencils ? 1 : 0, pt = t - c * pencils;
            const int pb = quot(pt, ax == 0 ? iny : inx), pa = pt - pb * m;
            double *v = a + c * kPlane + pa * sa + pb * sb;
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const int k = 4 * st + kq;
                const double x = k < len ? v[k * stride] : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qv[st], x, acc, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (kq + 4 * i < len && t0 + pn < NC * pencils) v[(kq + 4 * i) * stride] = acc[i];
        }
        __syncthreads();
        if (pass == 2) {
            for (int i = threadIdx.x; i < n; i += blockDim.x) {
                const int r = quot(i, inx), x = i - r * nx, z = quot(r, iny), y = r - z * ny, o = r * sy + x;
                const double lr = d.cx * eig[x] + d.cy * eig[kMgCoarseMax + y] + d.cz * eig[2 * kMgCoarseMax + z] + d.kre;
                const double li = d.kim, den = lr * lr + li * li;
                const double id = den == 0.0 ? 0.0 : 1.0 / den, wr = lr * id, wi = -li * id;
                const double vr = a[o];
                if constexpr (NC == 2) {
                    const double vi = a[kPlane + o];
                    a[o] = vr * wr - vi * wi;
                    a[kPlane + o] = vr * wi + vi * wr;
                } else {
                    a[o] = vr * wr;
                }
            }
            __syncthreads();
        }
    }
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int r = quot(i, inx), o = r * sy + i - r * nx;
        TO v;
        mg_from_c(make_double2(a[o], NC == 2 ? a[(NC - 1) * kPlane + o] : 0.0), v);
        u.st(i, v);
    }
}

// Level array of systems q0 .. q0 + count - 1 of a hierarchy.
template <typename S>
MgArr<S> lvl(void *base, const MgLevel &L, int q0) {
    return MgArr<S>{base ? (S *)base + (int64_t)q0 * L.n : nullptr, L.n, nullptr};
}

// Column capacities of the cycle kernels' workgroups (threads x columns per
// thread).
constexpr int kMgCaps[4] = {256, 512, 1024, 2048};

// The tile of a level: the smallest modelled time over the column capacities
// and the even splits of the axes.  `halo` is the (x, y) region's excess over
// the tile, `warm` the extra z steps of a chunk, `bufs` the LDS planes held.
// A step of a workgroup costs a latency (barrier, LDS round trip, the wait
// for the fetch two planes back) or, with enough columns resident on the
// compute unit, its columns' share of the bandwidth.  So large grids take
// large tiles and long chunks (little halo and warm-up), and small ones many
// small workgroups.  Measured at 320^3 (down / up, us): 2048 columns 148 / 140,
// 1024 columns 150 / 174, 512 200 / 168, 256 225 / 217; at 96^3 2048 columns
// 13 / 12, 256 columns 12 / 10; at 24^3 9 / 10 and 6 / 6.
MgPick mg_pick_tile(const MgLevel &L, int count, size_t elem, int halo, int warm, int bufs) {
    constexpr double kStep = 0.55, kCol = 0.0008;     // us; kCol per column of 4 bytes
    MgPick best;
    double best_cost = -1.0;
    best.cap = kMgCaps[0];
    best.count = count;
    for (int cols : kMgCaps) {
        const size_t lds = elem * cols * bufs;
        if (lds > 100 * 1024 || (elem == 16 && cols > 1024)) break;    // complex128: registers
        const int threads = cols >= 1024 ? 512 : 256;
        const int occ = std::max(1, std::min((int)(160 * 1024 / lds), 1536 / threads));
        for (int tx = 1; tx <= L.nx / 2; ++tx) {
            const int W = 2 * ((L.nx / 2 + tx - 1) / tx);
            if (W > 128) continue;
            if (W < 8 && tx > 1) break;
            if (tx > 1 && W * (tx - 1) >= L.nx) continue;          // an empty last tile
            const int hmax = (cols / (W + halo) - halo) & ~1;
            if (hmax < 2) continue;
            const int ty = (L.ny / 2 + hmax / 2 - 1) / (hmax / 2);
            const int H = 2 * ((L.ny / 2 + ty - 1) / ty);
            for (int tz = 1; tz <= L.nz / 2; ++tz) {
                const int zl = 2 * ((L.nz / 2 + tz - 1) / tz);
                if (tz > 1 && zl * (tz - 1) >= L.nz) continue;
                const double blocks = (double)tx * ty * tz * count;
                const double cu = std::min((double)occ, std::ceil(blocks / 256.0));
                const double waves = std::ceil(blocks / (256.0 * occ));
                const double step = std::max(kStep, cu * cols * kCol * (double)elem / 4.0);
                const double cost = waves * (zl + warm) * step;
                if (best_cost < 0.0 || cost < best_cost) {
                    best_cost = cost;
                    best.t = MgTile{W, H, zl, tx, ty, tz};
                    best.cap = cols;
                }
                if (zl <= 4) break;
            }
        }
    }
    return best;
}

// Systems of a launch for which the tile of a kernel with products is picked:
// four shifted systems on a grid (the density functional's batches), one real one.
constexpr int mg_dot_systems(size_t elem) { return elem == 16 ? 4 : 1; }

MgPick mg_pick_down(const MgLevel &L, int count, size_t elem) { return mg_pick_tile(L, count, elem, 5, 5, 6); }
MgPick mg_pick_up(const MgLevel &L, int count, size_t elem) { return mg_pick_tile(L, count, elem, 4, 4, 4); }

template <typename TF, typename S>
int launch_down(const MgLevel &L, const MgLevel &C, int count, double2 kappa, double omega, MgArr<const TF> f,
                MgArr<S> u, MgArr<S> cf, MgShift sh, hipStream_t s) {
    const MgPick pick = L.down[0].count == count   ? L.down[0]
                        : L.down[1].count == count ? L.down[1]
                                                   : mg_pick_down(L, count, sizeof(S));
    const MgTile t = pick.t;
    const MgDims d = dims_of(L, kappa), cd = dims_of(C, kappa);
    const dim3 grid(t.blocks() * count);
    switch (pick.cap) {
        case 256: hipLaunchKernelGGL((mg_down<TF, S, 256, 1>), grid, dim3(256), 0, s, d, cd, t, omega, f, u, cf, sh); break;
        case 512: hipLaunchKernelGGL((mg_down<TF, S, 256, 2>), grid, dim3(256), 0, s, d, cd, t, omega, f, u, cf, sh); break;
        case 1024: hipLaunchKernelGGL((mg_down<TF, S, 512, 2>), grid, dim3(512), 0, s, d, cd, t, omega, f, u, cf, sh); break;
        default:
            if constexpr (sizeof(S) <= 8)
                hipLaunchKernelGGL((mg_down<TF, S, 512, 4>), grid, dim3(512), 0, s, d, cd, t, omega, f, u, cf, sh);
    }
    OFDFT_CHECK_HIP(hipGetLastError());
    return OFDFT_OK;
}

template <class Dot, typename TF, typename S, typename TO>
int launch_up(const MgLevel &L, const MgLevel &C, int count, double2 kappa, double omega, MgArr<const TF> f,
              MgArr<const S> u, MgArr<const S> cu, MgArr<TO> z, MgShift sh, MgDot<Dot> dot, hipStream_t s) {
    // a system's products are summed in an order of its own, whatever it shares the launch with
    const MgPick pick = Dot::kSums               ? L.dot
                        : L.up[0].count == count ? L.up[0]
                        : L.up[1].count == count ? L.up[1]
                                                 : mg_pick_up(L, count, sizeof(S));
    const MgTile t = pick.t;
    if (Dot::kSums && t.blocks() > dot.cap) return OFDFT_INVALID_ARG;     // sized by mg_create
    const MgDims d = dims_of(L, kappa), cd = dims_of(C, kappa);
    const dim3 grid(t.blocks() * count);
    switch (pick.cap) {
        case 256: hipLaunchKernelGGL((mg_up<TF, S, TO, 256, 1, Dot>), grid, dim3(256), 0, s, d, cd, t, omega, f, u, cu, z, sh, dot); break;
        case 512: hipLaunchKernelGGL((mg_up<TF, S, TO, 256, 2, Dot>), grid, dim3(256), 0, s, d, cd, t, omega, f, u, cu, z, sh, dot); break;
        case 1024: hipLaunchKernelGGL((mg_up<TF, S, TO, 512, 2, Dot>), grid, dim3(512), 0, s, d, cd, t, omega, f, u, cu, z, sh, dot); break;
        default:
            if constexpr (sizeof(S) <= 8)
                hipLaunchKernelGGL((mg_up<TF, S, TO, 512, 4, Dot>), grid, dim3(512), 0, s, d, cd, t, omega, f, u, cu, z, sh, dot);
    }
    OFDFT_CHECK_HIP(hipGetLastError());
    return OFDFT_OK;
}

// V(2,2) cycle on level l >= 1 (arrays of S) of `count` systems from q0:
// f -> t (the coarsest level: f -> t by the exact solve).
template <typename S>
int vcycle_coarse(Multigrid &mg, int l, int q0, int count, double2 kappa, MgShift sh, hipStream_t s) {
    MgLevel &L = mg.lv[l];
    const MgArr<S> u = lvl<S>(L.u, L, q0), t = lvl<S>(L.t, L, q0);
    const MgArr<const S> f{(const S *)L.f + (int64_t)q0 * L.n, L.n, nullptr}, uc{u.base, u.stride, nullptr};
    if (l + 1 == (int)mg.lv.size()) {
        const MgDims d = dims_of(L, kappa);
        hipLaunchKernelGGL((mg_coarse_solve<S, S>), dim3(count), dim3(kMgCoarseThreads), 0, s, d, f, t, sh, mg.tab);
        OFDFT_CHECK_HIP(hipGetLastError());
        return OFDFT_OK;
    }
    MgLevel &C = mg.lv[l + 1];
    OFDFT_TRY((launch_down<S, S>(L, C, count, kappa, mg.omega, f, u, lvl<S>(C.f, C, q0), sh, s)));
    OFDFT_TRY(vcycle_coarse<S>(mg, l + 1, q0, count, kappa, sh, s));
    const MgArr<const S> ct{(const S *)C.t + (int64_t)q0 * C.n, C.n, nullptr};
    return launch_up<MgNoDot, S, S, S>(L, C, count, kappa, mg.omega, f, uc, ct, t, sh, {}, s);
}

// The whole cycle z = M f for `count` systems from q0 of the hierarchy: level
// 0 reads f and writes z in FP64 (TIO), its work arrays are S.  V(2,2), two
// kernels per level.  f, z, sh and dot address system q0 first.
template <typename TIO, typename S, class Dot = MgNoDot>
int vcycle(Multigrid &mg, int q0, int count, MgArr<const TIO> f, MgArr<TIO> z, double2 kappa, MgShift sh,
           hipStream_t s, Dot prod = {}) {
    MgLevel &L = mg.lv[0];
    if (mg.lv.size() == 1) {
        const MgDims d = dims_of(L, kappa);
        hipLaunchKernelGGL((mg_coarse_solve<TIO, TIO>), dim3(count), dim3(kMgCoarseThreads), 0, s, d, f, z, sh, mg.tab);
        OFDFT_CHECK_HIP(hipGetLastError());
        return OFDFT_OK;
    }
    const MgArr<S> u = lvl<S>(L.u, L, q0);
    const MgArr<const S> uc{u.base, u.stride, nullptr};
    MgLevel &C = mg.lv[1];
    const MgArr<S> cf = lvl<S>(C.f, C, q0);
    const MgArr<const S> ct{(const S *)C.t + (int64_t)q0 * C.n, C.n, nullptr};
    OFDFT_TRY((launch_down<TIO, S>(L, C, count, kappa, mg.omega, f, u, cf, sh, s)));
    OFDFT_TRY(vcycle_coarse<S>(mg, 1, q0, count, kappa, sh, s));
    const MgDot<Dot> dot{prod, mg.dpart + (int64_t)q0 * Multigrid::kDotSums * mg.dot_cap, mg.dctr + (int64_t)q0 * kArriveWords,
                         mg.dot_cap};
    return launch_up<Dot, TIO, S, TIO>(L, C, count, kappa, mg.omega, f, uc, ct, z, sh, dot, s);
}

}  // namespace

int mg_create(Multigrid &mg, const ofdft_grid &g, int elem_bytes, bool fp32, int groups) {
    mg_free(mg);
    if ((elem_bytes != 8 && elem_bytes != 16) || groups < 1) return OFDFT_INVALID_ARG;
    // no limits of these launches (which are one-dimensional): what is refused and
    // accepted here has been part of the interface since they had three dimensions
    if (((int64_t)g.nz + 3) / 4 * groups > 65535) {
        set_error("multigrid: %d systems of %d planes exceed one launch", groups, g.nz);
        return OFDFT_INVALID_ARG;
    }
    if (g.nz > 65535) {
        set_error("multigrid: nz = %d exceeds 65535", g.nz);
        return OFDFT_INVALID_ARG;
    }
    mg.elem = elem_bytes;
    mg.fp32 = fp32;
    mg.groups = groups;
    MgLevel L;
    L.nx = g.nx;
    L.ny = g.ny;
    L.nz = g.nz;
    L.cx = 1.0 / (g.hx * g.hx);
    L.cy = 1.0 / (g.hy * g.hy);
    L.cz = 1.0 / (g.hz * g.hz);
    for (;;) {
        L.n = (int64_t)L.nx * L.ny * L.nz;
        mg.lv.push_back(L);
        const bool small = L.nx <= kMgCoarseMax && L.ny <= kMgCoarseMax && L.nz <= kMgCoarseMax;
        if (small) break;
        if (L.nx % 2 || L.ny % 2 || L.nz % 2) {
            set_error("multigrid: grid %dx%dx%d cannot be halved down to %d per axis", g.nx, g.ny, g.nz,
                      kMgCoarseMax);
            mg.lv.clear();
            return OFDFT_INVALID_ARG;
        }
        L.nx /= 2;
        L.ny /= 2;
        L.nz /= 2;
        L.cx /= 4.0;
        L.cy /= 4.0;
        L.cz /= 4.0;
    }
    const size_t es = fp32 ? (size_t)elem_bytes / 2 : (size_t)elem_bytes;
    const int nlev = (int)mg.lv.size();
    for (int l = 0; l < nlev; ++l) {
        MgLevel &M = mg.lv[l];
        const size_t b = es * (size_t)M.n * (size_t)groups;
        // u: every level with a coarser one; f and t, the level's right-hand side
        // and solution: below the first (the caller's f and z there).  A
        // one-level hierarchy needs nothing.
        void **own[3];
        int count = 0;
        if (l + 1 < nlev) own[count++] = &M.u;
        if (l > 0) {
            own[count++] = &M.f;
            own[count++] = &M.t;
        }
        for (int k = 0; k < count; ++k) {
            void *p = nullptr;
            if (hipMalloc(&p, b) != hipSuccess) {
                (void)hipGetLastError();
                mg_free(mg);
                set_error("multigrid: out of device memory");
                return OFDFT_NO_MEMORY;
            }
            mg.allocs.push_back(p);
            *own[k] = p;
        }
    }
    for (int l = 0; l + 1 < nlev; ++l) {
        MgLevel &M = mg.lv[l];
        for (int k = 0; k < (groups > 1 ? 2 : 1); ++k) {
            M.down[k] = mg_pick_down(M, k ? groups : 1, es);
            M.up[k] = mg_pick_up(M, k ? groups : 1, es);
        }
    }
    if (nlev > 1) {              // reductions of the products in level 0's last kernel
        mg.lv[0].dot = mg_pick_up(mg.lv[0], mg_dot_systems((size_t)elem_bytes), es);
        mg.dot_cap = mg.lv[0].dot.t.blocks();
        const size_t bp = sizeof(double) * Multigrid::kDotSums * (size_t)mg.dot_cap * groups, bc = sizeof(unsigned int) * kArriveWords * (size_t)groups;
        void *p = nullptr;
        if (hipMalloc(&p, bp + bc) != hipSuccess) {
            (void)hipGetLastError();
            mg_free(mg);
            set_error("multigrid: out of device memory");
            return OFDFT_NO_MEMORY;
        }
        mg.allocs.push_back(p);
        mg.dpart = (double *)p;
        mg.dctr = (unsigned int *)((char *)p + bp);
        OFDFT_CHECK_HIP(hipMemset(mg.dctr, 0, bc));
    }
    // tables of the coarsest grid's exact solve
    const MgLevel &B = mg.lv.back();
    std::vector<double> tab(6 * kMgTab + 3 * kMgCoarseMax, 0.0);
    for (int ax = 0; ax < 3; ++ax) {
        const int len = ax == 0 ? B.nx : (ax == 1 ? B.ny : B.nz);
        for (int k = 0; k < len; ++k) {
            const double th = 2.0 * 3.14159265358979323846 / len;
            const double c = std::sqrt((k == 0 || 2 * k == len ? 1.0 : 2.0) / len);
            for (int j = 0; j < len; ++j) {
                const double w = 2 * k <= len ? c * std::cos(th * (k * j % len)) : c * std::sin(th * ((len - k) * j % len));
                tab[ax * kMgTab + k * kMgCoarseMax + j] = w;
                tab[(3 + ax) * kMgTab + j * kMgCoarseMax + k] = w;
            }
            tab[6 * kMgTab + ax * kMgCoarseMax + k] = k == 0 ? 0.0 : 2.0 - 2.0 * std::cos(th * k);
        }
    }
    void *p = nullptr;
    if (hipMalloc(&p, sizeof(double) * tab.size()) != hipSuccess) {
        (void)hipGetLastError();
        mg_free(mg);
        set_error("multigrid: out of device memory");
        return OFDFT_NO_MEMORY;
    }
    mg.allocs.push_back(p);
    mg.tab = (double *)p;
    if (hipMemcpy(p, tab.data(), sizeof(double) * tab.size(), hipMemcpyHostToDevice) != hipSuccess) {
        mg_free(mg);
        set_error("multigrid: table upload failed");
        return OFDFT_HIP_ERROR;
    }
    return OFDFT_OK;
}

void mg_free(Multigrid &mg) {
    for (void *p : mg.allocs) (void)hipFree(p);
    mg.allocs.clear();
    mg.lv.clear();
    mg.tab = nullptr;
    mg.dpart = nullptr;
    mg.dctr = nullptr;
    mg.dot_cap = 0;
}

int mg_apply(Multigrid &mg, const double *r, double *z, hipStream_t s, double kappa) {
    if (mg.lv.empty() || mg.elem != 8) return OFDFT_INVALID_ARG;
    ProfScope ps(K_MULTIGRID, mg_cycle_bytes(mg), s);
    const double2 k = make_double2(kappa, 0.0);
    const MgShift sh{nullptr, nullptr, 0, 0};
    const MgArr<const double> f{r, 0, nullptr};
    const MgArr<double> o{z, 0, nullptr};
    return mg.fp32 ? vcycle<double, float>(mg, 0, 1, f, o, k, sh, s)
                   : vcycle<double, double>(mg, 0, 1, f, o, k, sh, s);
}

int mg_apply_run(Multigrid &mg, const double *r, double *z, hipStream_t s, double kappa, const int *run) {
    if (mg.lv.empty() || mg.elem != 8) return OFDFT_INVALID_ARG;
    ProfScope ps(K_MULTIGRID, 0.0, s);      // bytes: the caller counts the cycles that ran
    const double2 k = make_double2(kappa, 0.0);
    const MgShift sh{nullptr, run, 0, 0};
    const MgArr<const double> f{r, 0, nullptr};
    const MgArr<double> o{z, 0, nullptr};
    return mg.fp32 ? vcycle<double, float>(mg, 0, 1, f, o, k, sh, s)
                   : vcycle<double, double>(mg, 0, 1, f, o, k, sh, s);
}

int mg_apply_run(Multigrid &mg, const double *r, double *z, hipStream_t s, double kappa, const int *run,
                 const MgUpdateDots &dots) {
    if (mg.lv.empty() || mg.elem != 8) return OFDFT_INVALID_ARG;
    ProfScope ps(K_MULTIGRID, 0.0, s);
    const double2 k = make_double2(kappa, 0.0);
    const MgShift sh{nullptr, run, 0, 0};
    const MgArr<const double> f{r, 0, nullptr};
    const MgArr<double> o{z, 0, nullptr};
    return mg.fp32 ? vcycle<double, float>(mg, 0, 1, f, o, k, sh, s, dots)
                   : vcycle<double, double>(mg, 0, 1, f, o, k, sh, s, dots);
}

int mg_apply_shifted(Multigrid &mg, int q, const double2 *r, double2 *z, const double *kappa, const int *run,
                     hipStream_t s) {
    if (mg.lv.empty() || mg.elem != 16 || !kappa || q < 0 || q >= mg.groups) return OFDFT_INVALID_ARG;
    const double2 k = make_double2(0.0, 0.0);
    const MgShift sh{kappa, run, 0, 0};
    const MgArr<const double2> f{r, 0, nullptr};
    const MgArr<double2> o{z, 0, nullptr};
    return mg.fp32 ? vcycle<double2, float2>(mg, q, 1, f, o, k, sh, s)
                   : vcycle<double2, double2>(mg, q, 1, f, o, k, sh, s);
}

int mg_apply_shifted(Multigrid &mg, int q, const double2 *r, double2 *z, const StepRho &rho, const double *kappa,
                     const int *run, hipStream_t s) {
    if (mg.lv.empty() || mg.elem != 16 || !kappa || q < 0 || q >= mg.groups) return OFDFT_INVALID_ARG;
    const double2 k = make_double2(0.0, 0.0);
    const MgShift sh{kappa, run, 0, 0};
    const MgArr<const double2> f{r, 0, nullptr};
    const MgArr<double2> o{z, 0, nullptr};
    return mg.fp32 ? vcycle<double2, float2>(mg, q, 1, f, o, k, sh, s, rho)
                   : vcycle<double2, double2>(mg, q, 1, f, o, k, sh, s, rho);
}

int mg_apply_shifted_group(Multigrid &mg, int count, const double2 *const *r, double2 *const *z, const StepRho &rho,
                           const double *kappa, int kstride, const int *run, int rstride, hipStream_t s) {
    if (mg.lv.empty() || mg.elem != 16 || !kappa || !r || !z || count < 1 || count > mg.groups)
        return OFDFT_INVALID_ARG;
    const double2 k = make_double2(0.0, 0.0);
    const MgShift sh{kappa, run, kstride, rstride};
    const MgArr<const double2> f{nullptr, 0, r};
    const MgArr<double2> o{nullptr, 0, z};
    return mg.fp32 ? vcycle<double2, float2>(mg, 0, count, f, o, k, sh, s, rho)
                   : vcycle<double2, double2>(mg, 0, count, f, o, k, sh, s, rho);
}

// Algorithmic bytes of one cycle.  Fine level: the downward half reads f and
// writes u and an eighth of an element (the restricted residual), the upward
// half reads f, u and an eighth (the coarse correction) and writes z.  Each
// coarser level moves 5.25 elements per point, and they hold 1/7 of the fine
// points in all.
double mg_cycle_bytes(const Multigrid &mg) {
    if (mg.lv.empty()) return 0.0;
    const double E = (double)mg.elem, e = mg.fp32 ? E / 2 : E;
    const double n = (double)mg.lv[0].n;
    if (mg.lv.size() == 1) return 2.0 * n * E;
    return n * (3.0 * E + 2.25 * e) + n / 7.0 * 5.25 * e;
}

// CG on the projected Poisson system preconditioned by the V-cycle (flexible
// CG form, which equals preconditioned CG for this fixed SPD operator).
// The start (residual, first cycle, rho = r^T z) runs with host reads; the
// iterations are driven from the device: alpha, the convergence test and
// beta are set by the last workgroup of the reductions in a device state
// (PDev), every pass returns at once when the solve is over, and blocks of
// kPcgBlock iterations are captured once in a HIP graph (x is read from the
// state, so one graph serves every solution array) and replayed with one host
// read per block.  Profiled runs of the classes launch the same kernels one by
// one.
//
// On large grids every pass is bound by memory, so p and x are not touched in
// each iteration: the stencil runs on z (A p = A z + beta A p_old), the last
// `ring` vectors z are kept, and every ring-th update brings p and x up to
// date from them (p = z_k + beta_k p, x += alpha_k p).  p^T A p =
// z^T A p + beta (z^T A p_old + beta p_old^T A p_old), and
// <z, r - r_old> = -alpha <z, A p>, so neither p nor r_old is needed for the
// scalars.  Bytes per point and iteration beside the cycle: 24 (stencil) + 24
// (r) + 8 (A p, read by the cycle's last kernel for the products) + 16 (p and x,
// ring 4) = 72; with p, x and r_old moved in each iteration and a pass for the
// products 120.  Measured, whole solves: the ring 320^3 17.8 -> 15.2 ms, 96^3
// 1.69 -> 1.59 ms; the products in the cycle 15.2 -> 14.1 and 1.61 -> 1.52 ms.
namespace {

constexpr int kPcgBlock = 4;
static_assert(kPcgBlock % kPcgRing == 0, "a captured block ends where the ring does (2 divides it, too)");
enum { P_RUN = 0, P_OK = 1, P_NONFINITE = 2, P_BREAKDOWN = 3, P_MAXIT = 4 };

struct EpiZAp {          // centre z: Ap = -L z + b Ap_old, <z, Ap>; p^T A p and alpha into the state
    double *__restrict__ Ap;
    PDev *D;
    int slot;
    double *partials;
    unsigned int *counter;
    double acc, b;
    double ao[4];
    __device__ bool skip() {
        b = D->b[slot];
        return D->done != P_RUN;
    }
    __device__ void pre(int q, int64_t i) { ao[q] = Ap[i]; }
    __device__ void point(int q, int64_t i, double c, double s) {
        const double a = ::fma(b, ao[q], -s);
        Ap[i] = a;
        acc = ::fma(c, a, acc);
    }
    __device__ void finish(int block, int nblocks, double *scratch) {
        double x[1] = {acc};
        block_sum<1>(x, scratch);
        double t[1];
        if (reduce_grid<1>(x, partials, nblocks, block, counter, scratch, t)) {
            const double pAp = t[0] + b * ::fma(b, D->pAp, D->zAp), rz = D->rz;
            D->pAp = pAp;
            D->n_ap += 1;
            if (!isfinite(pAp) || !isfinite(rz)) D->done = P_NONFINITE;
            else if (!(pAp > 0.0) || !(rz > 0.0)) D->done = P_BREAKDOWN;
            else D->a[slot] = rz / pAp;
        }
    }
};

// r -= a Ap; {<r,r>}; with Ring > 0 (in the ring's last slot) also p and x.
template <int Ring>
struct PcgStepOp {
    static constexpr int kClass = K_CG_UPDATE;
    static constexpr int kBytes = 0;     // counted from the passes that did work
    static constexpr int kSlots = Ring ? Ring : 1;
    double *r;
    const double *Ap;
    double *p;
    const double *z[kSlots];
    PDev *D;
    int slot;
    double *x;
    double a[kSlots], b[kSlots], al;
    bool have;                           // p holds a direction
    __device__ bool skip() const { return D->done != P_RUN; }
    __device__ void prepare() {
        al = D->a[slot];
        if constexpr (Ring > 0) {
            x = D->x;
            have = D->iters >= Ring;
            for (int k = 0; k < Ring; ++k) {
                a[k] = D->a[k];
                b[k] = D->b[k];
            }
        }
    }
    __device__ void operator()(int64_t i, double (&acc)[1]) const {
        const double rn = ::fma(-al, Ap[i], r[i]);
        if constexpr (Ring > 0) {
            double zv[Ring];
            for (int k = 0; k < Ring; ++k) zv[k] = z[k][i];
            double pv = have ? p[i] : 0.0, xv = x[i];
            for (int k = 0; k < Ring; ++k) {
                pv = ::fma(b[k], pv, zv[k]);
                xv = ::fma(a[k], pv, xv);
            }
            p[i] = pv;
            x[i] = xv;
        }
        r[i] = rn;
        acc[0] = ::fma(rn, rn, acc[0]);
    }
};
struct FinStepP {
    PDev *D;
    __device__ void operator()(const double (&t)[1]) const {
        const double r2 = t[0];
        D->r2 = r2;
        D->iters += 1;
        D->n_step += 1;
        if (!isfinite(r2)) D->done = P_NONFINITE;
        else if (r2 <= D->tol2) D->done = P_OK;
        else if (D->iters >= D->maxit) D->done = P_MAXIT;
    }
};

struct PcgFinishOp {     // x of a solve that stopped between two updates of x: the ring's first cnt directions
    static constexpr int kClass = K_CG_UPDATE;
    static constexpr int kBytes = 0;
    const double *p;
    const double *z[kPcgRing];
    const PDev *D;
    int cnt, have;
    double *x;
    __device__ bool skip() const { return false; }
    __device__ void prepare() { x = D->x; }
    __device__ void operator()(int64_t i, double (&)[1]) const {
        double pv = have ? p[i] : 0.0, xv = x[i];
#pragma unroll
        for (int k = 0; k < kPcgRing; ++k)
            if (k < cnt) {
                pv = ::fma(D->b[k], pv, z[k][i]);
                xv = ::fma(D->a[k], pv, xv);
            }
        x[i] = xv;
    }
};

struct PcgDotsOp {       // PcgRho's sums after a one-level cycle
    static constexpr int kClass = K_CG_UPDATE;
    static constexpr int kBytes = 0;
    const double *z, *r;
    PcgRho rho;
    __device__ bool skip() const { return rho.D->done != P_RUN; }
    __device__ void prepare() {}
    __device__ void operator()(int64_t i, double (&acc)[2]) const { PcgRho::point(acc, z[i], r[i], rho.Ap[i]); }
};
struct PcgDotsFin {
    PcgRho rho;
    __device__ void operator()(const double (&t)[2]) const { rho.finish(0, t); }
};

// One iteration, its z in ring slot `slot`.
int pcg_iteration(ofdft_poisson *s, int slot, hipStream_t st) {
    const ofdft_grid &g = s->g;
    const int64_t n = npoints(g);
    PDev *D = (PDev *)s->pdev;
    const int ring = s->mg_ring, next = (slot + 1) % ring;
    double *r = s->r, *p = s->pA, *Ap = s->Ap, *const *z = s->mg_z;
    {
        ProfScope ps(K_CG_STENCIL, 0.0, st);
        OFDFT_TRY(launch_stencil<double>(g, s->coef, LoadPlain<double>{z[slot]},
                                         EpiZAp{Ap, D, slot, s->rb.partials, s->rb.counter, 0.0, 0.0, {}}, st));
    }
    if (next) {
        OFDFT_TRY((launch_reduce<1>(n, PcgStepOp<0>{r, Ap, nullptr, {nullptr}, D, slot}, FinStepP{D}, s->rb, st)));
    } else if (ring == 2) {
        OFDFT_TRY((launch_reduce<1>(n, PcgStepOp<2>{r, Ap, p, {z[0], z[1]}, D, slot}, FinStepP{D}, s->rb, st)));
    } else {
        static_assert(kPcgRing == 4, "one entry per slot below");
        OFDFT_TRY((launch_reduce<1>(n, PcgStepOp<4>{r, Ap, p, {z[0], z[1], z[2], z[3]}, D, slot}, FinStepP{D},
                                    s->rb, st)));
    }
    const PcgRho rho{Ap, D, slot, next};
    if (!mg_forms_dots(*s->mg)) {
        OFDFT_TRY(mg_apply_run(*s->mg, r, z[next], st, 0.0, &D->done));
        return launch_reduce<2>(n, PcgDotsOp{z[next], r, rho}, PcgDotsFin{rho}, s->rb, st);
    }
    ProfScope ps(K_MULTIGRID, 0.0, st);      // bytes: counted with the cycles that ran
    const MgShift sh{nullptr, &D->done, 0, 0};
    const MgArr<const double> f{r, 0, nullptr};
    const MgArr<double> o{z[next], 0, nullptr};
    const double2 k0 = make_double2(0.0, 0.0);
    return s->mg->fp32 ? vcycle<double, float>(*s->mg, 0, 1, f, o, k0, sh, st, rho)
                       : vcycle<double, double>(*s->mg, 0, 1, f, o, k0, sh, st, rho);
}

int pcg_graph(ofdft_poisson *s) {
    if (s->mggraph) return OFDFT_OK;
    if (!s->mgcap) OFDFT_CHECK_HIP(hipStreamCreateWithFlags(&s->mgcap, hipStreamNonBlocking));
    hipGraph_t graph = nullptr;
    OFDFT_CHECK_HIP(hipStreamBeginCapture(s->mgcap, hipStreamCaptureModeThreadLocal));
    prof_suspend(true);
    int rc = OFDFT_OK;
    for (int k = 0; k < kPcgBlock && rc == OFDFT_OK; ++k) rc = pcg_iteration(s, k % s->mg_ring, s->mgcap);
    prof_suspend(false);
    const hipError_t e = hipStreamEndCapture(s->mgcap, &graph);
    if (rc != OFDFT_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return rc;
    }
    OFDFT_CHECK_HIP(e);
    const hipError_t ei = hipGraphInstantiate(&s->mggraph, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    OFDFT_CHECK_HIP(ei);
    return OFDFT_OK;
}

}  // namespace

int poisson_solve_mg(ofdft_poisson *s, double *x, double rel_tol, int max_iter, ofdft_solve_stats &stats,
                     hipStream_t st) {
    const ofdft_grid &g = s->g;
    const int64_t n = npoints(g);
    double *r = s->r, *z = s->z;
    double *tot = s->totals + 8, *th = s->totals_host + 8;
    auto sync_tot = [&](int count) -> int {
        OFDFT_CHECK_HIP(hipMemcpyAsync(th, tot, sizeof(double) * count, hipMemcpyDeviceToHost, st));
        OFDFT_CHECK_HIP(hipStreamSynchronize(st));
        return OFDFT_OK;
    };
    OFDFT_CHECK_HIP(hipMemcpyAsync(s->totals_host, s->totals, sizeof(double) * 4, hipMemcpyDeviceToHost, st));
    OFDFT_CHECK_HIP(hipStreamSynchronize(st));
    const double g2 = s->totals_host[3];
    const double tol2 = rel_tol * rel_tol * g2;
    OFDFT_TRY(residual_pass<double>(g, s->coef, x, s->gp, r, tot, s->rb, st));
    OFDFT_TRY(sync_tot(2));
    const double r2 = th[1];
    stats.iters = 0;
    if (!std::isfinite(r2)) return OFDFT_NONFINITE;
    if (r2 <= tol2) return OFDFT_OK;
    if (max_iter <= 0) return OFDFT_NOT_CONVERGED;
    OFDFT_TRY(mg_apply(*s->mg, r, z, st));
    OFDFT_TRY((launch_reduce<2>(n, FcgDotsOp{z, r, r}, StoreTotals<2>{tot}, s->rb, st)));
    OFDFT_TRY(sync_tot(2));
    // the first iteration's beta is 0, and its A p_old has to be finite
    OFDFT_CHECK_HIP(hipMemsetAsync(s->Ap, 0, sizeof(double) * n, st));
    if (!s->pdev) {
        OFDFT_CHECK_HIP(hipMalloc(&s->pdev, sizeof(PDev)));
        OFDFT_CHECK_HIP(hipHostMalloc(&s->pdev_h, sizeof(PDev), hipHostMallocDefault));
    }
    PDev *Dh = (PDev *)s->pdev_h;
    *Dh = PDev{};
    Dh->x = x;
    Dh->rz = th[1];
    Dh->tol2 = tol2;
    Dh->maxit = max_iter;
    OFDFT_CHECK_HIP(hipMemcpyAsync(s->pdev, Dh, sizeof(PDev), hipMemcpyHostToDevice, st));
    auto read_state = [&]() -> int {
        OFDFT_CHECK_HIP(hipMemcpyAsync(Dh, s->pdev, sizeof(PDev), hipMemcpyDeviceToHost, st));
        OFDFT_CHECK_HIP(hipStreamSynchronize(st));
        return OFDFT_OK;
    };
    const bool eager = !s->use_graphs || prof_timed(K_CG_STENCIL) || prof_timed(K_CG_UPDATE) ||
                       prof_timed(K_MULTIGRID);
    if (eager) {
        for (int k = 0; k <= max_iter; ++k) {
            OFDFT_TRY(pcg_iteration(s, k % s->mg_ring, st));
            OFDFT_TRY(read_state());
            if (Dh->done != P_RUN) break;
        }
    } else {
        OFDFT_TRY(pcg_graph(s));
        for (int k = 0; k <= max_iter; k += kPcgBlock) {
            OFDFT_CHECK_HIP(hipGraphLaunch(s->mggraph, st));
            OFDFT_TRY(read_state());
            if (Dh->done != P_RUN) break;
        }
    }
    const double nd = (double)n;
    const int ring = s->mg_ring, owed = Dh->iters % ring, flushes = Dh->iters / ring;
    if (owed) {
        PcgFinishOp fin{s->pA, {}, (const PDev *)s->pdev, owed, Dh->iters >= ring, nullptr};
        for (int k = 0; k < owed; ++k) fin.z[k] = s->mg_z[k];
        OFDFT_TRY((launch_reduce<1>(n, fin, NoFin{}, s->rb, st)));
        prof_add(K_CG_UPDATE, nd * 8.0 * (owed + (Dh->iters >= ring ? 3 : 2)), 0);
    }
    // stencil: read z, Ap_old, write Ap; update: read r, Ap, write r, every
    // ring-th one reads the ring, p, x and writes p, x (the first reads no p);
    // products: Ap in the cycle, after a one-level one z, r, Ap
    prof_add(K_CG_STENCIL, nd * 24.0 * Dh->n_ap, eager ? 0 : Dh->n_ap);
    prof_add(K_CG_UPDATE, nd * 8.0 * (3.0 * Dh->n_step + (mg_forms_dots(*s->mg) ? 0.0 : 3.0) * Dh->n_dots + (flushes ? (ring + 4.0) * flushes - 1.0 : 0.0)),
             eager ? 0 : Dh->n_step + (mg_forms_dots(*s->mg) ? 0 : Dh->n_dots));
    const double extra = mg_forms_dots(*s->mg) ? 8.0 * nd : 0.0;
    prof_add(K_MULTIGRID, (mg_cycle_bytes(*s->mg) + extra) * Dh->n_dots, eager ? 0 : Dh->n_dots);
    stats.iters = Dh->iters;
    switch (Dh->done) {
        case P_OK: return OFDFT_OK;
        case P_NONFINITE: return OFDFT_NONFINITE;
        case P_BREAKDOWN: return OFDFT_BREAKDOWN;
        default: return OFDFT_NOT_CONVERGED;
    }
}

}  // namespace ofdft

using namespace ofdft;

// z = M r for a multigrid solver (for inspection and for callers that build
// their own Krylov loop around the preconditioner).
extern "C" int ofdft_poisson_apply_preconditioner(ofdft_poisson *s, const double *r, double *z,
                                                  void *stream) {
    if (!s || !r || !z || r == z || !s->mg) {
        set_error("ofdft_poisson_apply_preconditioner: multigrid solver and distinct r, z required");
        return OFDFT_INVALID_ARG;
    }
    return mg_apply(*s->mg, r, z, (hipStream_t)stream);
}
