// Conjugate gradients of a grid that fits one workgroup: the whole iteration
// of cg.hpp (same recurrences, same tests, CgState in and out) in one launch.
//
// A 16^3 solve is 64 iterations of 4096 points: two launches per iteration
// take 14 us, nearly all of it launch and reduction latency.  Here p lives in
// LDS, x, r and A p in the registers of 1024 threads, and an iteration is two
// block reductions and three barriers.  A thread owns KZ consecutive planes of
// one (x, y) column.  Bound by LDS reads (24 + (KZ + 12) / KZ per point); rows
// of p carry a 6-wide periodic halo in x, so x neighbours are constant offsets,
// y offsets are computed once per solve, and z values are read once per column.
// Measured at 16^3, FP64, to 1e-10: 0.92 ms with two launches per iteration,
// 0.48 so (5.4 us per iteration).  A launch runs kTinyIters iterations at most
// and p is kept for the next, so that no solve, also one whose tolerance cannot
// be met, holds the stream for longer than some milliseconds.
#pragma once

#include "cg.hpp"

namespace ofdft {

constexpr int kTinyThreads = 1024;
constexpr int kTinyMinAxis = 6;          // one periodic wrap per offset
constexpr size_t kTinyLds = 140 * 1024;
constexpr int kTinyIters = 512;          // per launch: 3 ms at 16^3, 5 ms at most

// Planes per thread (4 or 8) if the grid fits one workgroup, else 0.  1024
// threads leave 128 registers: of a kernel of 4 planes 50 spill, of 8 180.  Per
// iteration to 1e-10, so and with two launches on bricks: FP64 4096 points 7.9 /
// 17.0 us, 4608 14.2 / 14.5, 5120 14.1 / 14.4, 6144 14.8 / 14.0, 8192 15.3 / 14.6; FP32
// 5120 11.5 / 17.1, 8192 12.5 / 16.4.  So FP64 grids of over 6000 points run two
// launches where their axes admit bricks (8 x 32 x 32, which does not: 15.2 / 23.0).
inline int tiny_planes(const ofdft_grid &g, size_t elem) {
    if (g.nx < kTinyMinAxis || g.ny < kTinyMinAxis || g.nz < kTinyMinAxis) return 0;
    if ((int64_t)g.nx * g.ny * g.nz > 8 * kTinyThreads) return 0;
    if ((size_t)(g.nx + 2 * kMaxRadius) * g.ny * g.nz * elem > kTinyLds) return 0;
    const bool bricks = g.nx >= kBrickMinAxis && g.ny >= kBrickMinAxis && g.nz >= kBrickMinAxis;
    if (elem == 8 && bricks && (int64_t)g.nx * g.ny * g.nz > 6000) return 0;
    for (int kz : {4, 8})
        if (g.nx * g.ny * ((g.nz + kz - 1) / kz) <= kTinyThreads) return kz;
    return 0;
}

// Sum over the workgroup, the result in every thread; `scratch` holds 17 doubles.
__device__ inline double tiny_sum(double x, double *scratch) {
    x = wave_sum(x);
    __syncthreads();                     // the previous sum has been read
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = x;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kTinyThreads / 64; ++i) s += scratch[i];
    return s;
}

template <typename T, int KZ, bool Resume>
__global__ void __launch_bounds__(kTinyThreads)
cg_tiny_kernel(int nx, int ny, int nz, Coef<typename VT<T>::S> w, T *__restrict__ x, T *__restrict__ r,
               T *__restrict__ pkeep, CgState *st) {
    using S = typename VT<T>::S;
    constexpr int R = kMaxRadius;
    extern __shared__ __align__(16) unsigned char tiny_lds[];
    T *const p = reinterpret_cast<T *>(tiny_lds);        // [nz][ny][nx + 12]
    __shared__ double scratch[kTinyThreads / 64 + 1];
    CgState s = *st;
    if (s.done != CG_RUNNING) return;
    const int P = nx + 2 * R, nxy = nx * ny, SL = P * ny;
    const int zg = threadIdx.x / nxy, col = threadIdx.x - zg * nxy;
    const int z0 = zg * KZ, cy = col / nx, cx = col - cy * nx;
    const int planes = min(KZ, nz - z0);                 // <= 0: the thread owns nothing
    const int row = cy * P + cx + R;                     // of plane 0
    int yo[2 * R + 1];                                   // offsets of rows cy - 6 .. cy + 6
#pragma unroll
    for (int j = 0; j < 2 * R + 1; ++j) {
        int yy = cy + j - R;
        yy = yy < 0 ? yy + ny : (yy >= ny ? yy - ny : yy);
        yo[j] = (yy - cy) * P;
    }
    // image of this column in the row's halo (cells -6 .. -1 and nx .. nx + 5)
    const int img = cx < R ? nx : (cx >= nx - R ? -nx : 0);
    const int img2 = cx < R && cx >= nx - R ? -nx : 0;   // a short row: on both sides
    T xv[KZ], rv[KZ], pv[KZ], av[KZ];
#pragma unroll
    for (int k = 0; k < KZ; ++k) {
        const bool own = k < planes;
        const int64_t i = (int64_t)(z0 + k) * nxy + col;
        xv[k] = own ? x[i] : T(0);
        rv[k] = own ? r[i] : T(0);
        pv[k] = Resume && own ? pkeep[i] : T(0);
        av[k] = T(0);
    }
    S beta = Resume ? (S)s.beta : S(0);
    const int maxit = s.maxit, cap = min(maxit, s.iter + kTinyIters);
    s.maxit = cap;                                       // one test serves the launch's cap and the solve's
    while (s.done == CG_RUNNING) {
        // p = r + beta p_old (first iteration: p = r)
#pragma unroll
        for (int k = 0; k < KZ; ++k)
            if (k < planes) {
                pv[k] = s.first ? rv[k] : VT<T>::fma(beta, pv[k], rv[k]);
                T *c = p + (z0 + k) * SL + row;
                c[0] = pv[k];
                if (img) c[img] = pv[k];
                if (img2) c[img2] = pv[k];
            }
        __syncthreads();
        double acc = 0.0;
        if (planes > 0) {
            T q[KZ + 2 * R];                             // planes z0 - 6 .. z0 + KZ + 5 of the column
#pragma unroll
            for (int j = 0; j < KZ + 2 * R; ++j) {
                int z = z0 + j - R;
                z = z < 0 ? z + nz : z;
                z = z >= nz ? z - nz : z;
                z = z >= nz ? z - nz : z;                // past a short last group: any plane
                q[j] = p[z * SL + row];
            }
#pragma unroll
            for (int k = 0; k < KZ; ++k)
                if (k < planes) {
                    const T *c = p + (z0 + k) * SL + row;
                    T sum = VT<T>::mul(w.c0, q[k + R]);
#pragma unroll
                    for (int d = 1; d <= R; ++d) {
                        sum = VT<T>::fma(w.wx[d], VT<T>::add(c[d], c[-d]), sum);
                        sum = VT<T>::fma(w.wy[d], VT<T>::add(c[yo[R + d]], c[yo[R - d]]), sum);
                        sum = VT<T>::fma(w.wz[d], VT<T>::add(q[k + R + d], q[k + R - d]), sum);
                    }
                    av[k] = VT<T>::mul(S(-1), sum);
                    acc = ::fma((double)pv[k], (double)av[k], acc);
                }
        }
        const double pAp = tiny_sum(acc, scratch);
        s.pAp = pAp;
        if (!isfinite(pAp)) {
            s.done = CG_NONFINITE;
            break;
        }
        if (!(pAp > 0.0)) {
            s.done = CG_BREAKDOWN;
            break;
        }
        s.alpha = s.rr / pAp;
        const S alpha = (S)s.alpha;
        acc = 0.0;
#pragma unroll
        for (int k = 0; k < KZ; ++k)
            if (k < planes) {
                xv[k] = VT<T>::fma(alpha, pv[k], xv[k]);
                rv[k] = VT<T>::fma(-alpha, av[k], rv[k]);
                acc = ::fma((double)rv[k], (double)rv[k], acc);
            }
        const double rr = tiny_sum(acc, scratch);
        s.beta = rr / s.rr;
        s.rr = rr;
        s.first = 0;
        s.iter += 1;
        if (!isfinite(rr)) s.done = CG_NONFINITE;
        else if (rr <= s.tol2) s.done = CG_CONVERGED;
        else if (s.iter >= s.maxit) s.done = CG_MAXIT;
        beta = (S)s.beta;
    }
#pragma unroll
    for (int k = 0; k < KZ; ++k)
        if (k < planes) {
            const int64_t i = (int64_t)(z0 + k) * nxy + col;
            x[i] = xv[k];
            r[i] = rv[k];
        }
    if (s.done == CG_MAXIT && cap < maxit) {             // p for the next launch
        s.done = CG_RUNNING;
        for (int k = 0; k < planes && k < KZ; ++k) pkeep[(int64_t)(z0 + k) * nxy + col] = p[(z0 + k) * SL + row];
    }
    s.maxit = maxit;
    if (threadIdx.x == 0) *st = s;
}

template <typename T>
inline int launch_cg_tiny(const ofdft_grid &g, int kz, const Coef<typename VT<T>::S> &c, T *x, T *r, T *p,
                          CgState *st, bool resume, hipStream_t s) {
    const size_t lds = (size_t)(g.nx + 2 * kMaxRadius) * g.ny * g.nz * sizeof(T);
    auto kern = kz == 4 ? (resume ? cg_tiny_kernel<T, 4, true> : cg_tiny_kernel<T, 4, false>)
                        : (resume ? cg_tiny_kernel<T, 8, true> : cg_tiny_kernel<T, 8, false>);
    hipLaunchKernelGGL(kern, dim3(1), dim3(kTinyThreads), lds, s, g.nx, g.ny, g.nz, c, x, r, p, st);
    OFDFT_CHECK_HIP(hipGetLastError());
    return OFDFT_OK;
}

}  // namespace ofdft
