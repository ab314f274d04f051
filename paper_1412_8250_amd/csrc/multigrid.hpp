// Geometric multigrid preconditioner for the periodic Poisson solve (the
// real-space preconditioner the paper's conclusion calls for, Section 5.5).
//
// M approximates the inverse of the 12th-order -L_h (+ kappa for the shifted
// systems) with one V(nu, nu) cycle of the second-order 7-point operator
// (+ kappa): damped Jacobi smoothing, full
// weighting restriction (R = P^T / 8), trilinear prolongation, every axis
// halved per level, and an exact DFT solve on the coarsest grid (at most 16
// points per axis).  The cycle is a fixed linear operator, symmetric and
// positive definite on zero-mean vectors (complex symmetric for a complex
// shift), so CG (COCG) preconditioned by it converges at a rate set by the
// spectral equivalence of the two operators, independent of the grid size.
#pragma once

#include <vector>

#include "common.hpp"

namespace ofdft {

struct StepRho;

// Launch geometry of the two cycle kernels of a level: a workgroup owns a
// W x H tile of (x, y) (both even) and marches along z over zl planes (even);
// tiles in x, y and z of one system, the systems of a launch one after
// another.
struct MgTile {
    int W, H, zl;
    int tx, ty, tz;
    __host__ __device__ int blocks() const { return tx * ty * tz; }
};

// The tile picked for launches of `count` systems and its column capacity.
struct MgPick {
    MgTile t{};
    int cap = 0, count = 0;
};

struct MgLevel {
    int nx = 0, ny = 0, nz = 0;
    double cx = 0, cy = 0, cz = 0;   // 1 / h_a^2
    int64_t n = 0;
    void *u = nullptr, *t = nullptr, *f = nullptr;   // element type of the levels
    // tiles of launches of one system and of all of the hierarchy's (searched in
    // every launch that is not replayed they cost the host 65 us a cycle at 512^3:
    // 100 where it is 35)
    MgPick down[2], up[2];
    MgPick dot;                      // the upward kernel that forms products
};

struct Multigrid {
    std::vector<MgLevel> lv;
    static constexpr int nu = 2; // Jacobi sweeps before and after the coarse correction
    double omega = 0.8;          // Jacobi damping
    int elem = 8;                // input / output element bytes: 8 (FP64) or 16 (complex128)
    bool fp32 = true;            // level arrays and their arithmetic in FP32 (else FP64)
    int groups = 1;              // systems whose level arrays the hierarchy holds (same grid)
    double *dpart = nullptr;     // partial sums (kDotSums dot_cap per system) and arrival counters of the products
    unsigned int *dctr = nullptr;
    int dot_cap = 0;
    const double *tab = nullptr; // coarsest grid: basis matrices and eigenvalues (device)
    std::vector<void *> allocs;
    static constexpr int kDotSums = 5;   // products per launch at most
};

constexpr int kMgCoarseMax = 16;     // coarsest grid: at most this many points per axis

// Hierarchy for grid g, applied to FP64 (elem_bytes 8) or complex128 (16)
// vectors; the level arrays (and the arithmetic on them) are FP32 / complex64
// when fp32 is set: the cycle then reads r and writes z in FP64 but is a fixed
// linear operator only to FP32 rounding, which the flexible and preconditioned
// Krylov loops here tolerate without extra iterations.  Every axis is halved
// while all are even and one exceeds kMgCoarseMax; INVALID_ARG if the
// coarsest grid would be larger than that.
// `groups` systems of this grid get level arrays of their own (system q's
// part of a level array starts q * n elements in), so that one launch per
// kernel can run the cycles of all of them.
int mg_create(Multigrid &mg, const ofdft_grid &g, int elem_bytes, bool fp32, int groups = 1);
void mg_free(Multigrid &mg);
// z = M r for -Delta + kappa, kappa >= 0 real (device FP64 arrays of the fine
// grid; z must not alias r).
int mg_apply(Multigrid &mg, const double *r, double *z, hipStream_t s, double kappa = 0.0);
// The same cycle, every kernel returning at once while *run != 0 (device
// flag, for cycles inside captured blocks of an iteration that may be over).
int mg_apply_run(Multigrid &mg, const double *r, double *z, hipStream_t s, double kappa, const int *run);
// The same with the density update's products <u,z>, <r,z>, <r_prev,z>, <u,r>,
// <u,r_prev> (the third and the last 0 while *q is 0) reduced into dots[0..4]
// by the last kernel, which then adds 1 to *count (if mg_forms_dots).
struct MgUpdateDots {
    static constexpr int kSums = 5;
    static constexpr bool kExtra = true;
    using Extra = double2;
    const double *u, *r_prev;
    const int *q;
    double *dots;
    int *count;
    bool have;
    __device__ void prepare() { have = *q > 0; }
    __device__ double2 extra(int64_t i) const {
        return make_double2(GPtr<double>(u)[i], have ? GPtr<double>(r_prev)[i] : 0.0);
    }
    __device__ static void point(double (&acc)[5], double z, double r, double2 e) {
        acc[0] = ::fma(e.x, z, acc[0]);
        acc[1] = ::fma(r, z, acc[1]);
        acc[2] = ::fma(e.y, z, acc[2]);
        acc[3] = ::fma(e.x, r, acc[3]);
        acc[4] = ::fma(e.x, e.y, acc[4]);
    }
    __device__ void finish(int, const double (&t)[5]) const {
        for (int k = 0; k < 5; ++k) dots[k] = t[k];
        *count += 1;
    }
};
int mg_apply_run(Multigrid &mg, const double *r, double *z, hipStream_t s, double kappa, const int *run,
                 const MgUpdateDots &dots);
// z = M r for -Delta + kappa (complex128 arrays).  kappa points to device
// memory holding {Re, Im} and is read by every launch, so a captured launch
// sequence follows later changes of the shift; if `run` is given, every
// kernel returns at once unless *run == 0 (a converged system of a batch).
// Not accounted in the profile (the caller accounts cycles).
// System q of the hierarchy's group does the cycle.
int mg_apply_shifted(Multigrid &mg, int q, const double2 *r, double2 *z, const double *kappa, const int *run,
                     hipStream_t s);
// The same, the last kernel also reducing the products of rho (if
// mg_forms_dots; else they are the caller's).
int mg_apply_shifted(Multigrid &mg, int q, const double2 *r, double2 *z, const StepRho &rho, const double *kappa,
                     const int *run, hipStream_t s);
// Whether the cycle's last kernel can form products of z: a hierarchy of more than one level.
inline bool mg_forms_dots(const Multigrid &mg) { return mg.lv.size() > 1; }
// The cycles of systems 0 .. count-1 of the group in one launch per kernel:
// system q reads r[q], writes z[q] (device tables of device pointers), its
// shift at kappa + q kstride and its run flag at run + q rstride (run may be
// null); rho as above, of system 0.  Not accounted in the profile.
int mg_apply_shifted_group(Multigrid &mg, int count, const double2 *const *r, double2 *const *z, const StepRho &rho,
                           const double *kappa, int kstride, const int *run, int rstride, hipStream_t s);
// Algorithmic HBM bytes of one cycle (products of r and z come with it).
double mg_cycle_bytes(const Multigrid &mg);

}  // namespace ofdft
