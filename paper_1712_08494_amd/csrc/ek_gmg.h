// Multigrid hierarchy with per-axis coarsening (ek_gmg.hip).  Not part of the public ABI.
#pragma once

#include <cstdint>
#include <vector>

#include "ek_internal.h"

namespace ek {

constexpr int kGMaxLevels = 16;
constexpr size_t kGmgLds = 160 * 1024;  // LDS of one workgroup
constexpr int kDirect = 32;             // cells of the coarsest grid at most: solved by its inverse
constexpr unsigned kSmallMost = 4096;   // sites of a lattice solved in one workgroup at most

// A coarse grid: cells per axis, and where its axis tables start: `of` indexes the tables
// over the cells of the finer grid (pn, w), `oc` those over its own cells (first, ratio).
struct GLevelDesc {
    int d[3];
    unsigned n;
    int lead;  // leading axes of one cell
    int of[3], oc[3];
};

// Host hierarchy, finest coarse grid first.
struct GHier {
    std::vector<GLevelDesc> levels;
    std::vector<uint32_t> pn;   // per fine cell of an axis: parent | neighbour towards the cell << 16
    std::vector<float> w;       // its interpolation weight on the neighbour
    std::vector<int> first;     // first child of each cell, and the end
    std::vector<float> ratio;   // fine over coarse centre distance at the face towards the next cell
};
void gmg_hierarchy(const int (&dims)[3], const bool (&periodic)[3], GHier& H);

// Device copies of the axis tables.
struct GTab {
    const uint32_t* pn;
    const float* w;
    const int* first;
    const float* ratio;
};

// A grid held in LDS: its axes, and the compact axes (ex, ey, ez) without leading ones of
// one cell, in which cells are coloured and rows evaluated.
struct GLds {
    int nx, ny, nz, ex, ey, ez, n, lead, off;
    int of[3], oc[3];
    float inv_hx, inv_ey, inv_nx, inv_ny;
};
struct GSub {
    int nl, cells, npn, nfirst;
    int pn0, first0;  // where its tables start in the hierarchy's
    GLds L[kGMaxLevels];
};
GSub gmg_sub(const GHier& H, int first, bool from_lattice);
int gmg_tail_first(const GHier& H);
size_t gmg_rows_bytes(const GSub& G);  // what launch_g_tail_build leaves for launch_g_tail
bool gmg_small_fits(const GSub& G, unsigned ndomain);

// V-cycle shape: sweeps on the lattice and on the coarse grids before and after the
// correction, relaxation (the coarsest grid is solved by its inverse).
struct GShape {
    int fine_pre, fine_post, pre, post;
    double omega;
};

// Solver state of the single-workgroup solve, doubles on the device at ctl: the adaptive
// warm start (last start residuals of orders 2 and 3, the order in use, steps since the
// other was probed, steps taken) and the record of the solves since the host last read it.
constexpr int kCtlRel0 = 0, kCtlOrder = 2, kCtlSince = 3, kCtlSteps = 4, kCtlNoConv = 5, kCtlIters = 6, kCtlTotal = 7,
              kCtlRel = 8, kCtlRelStart = 9, kCtlRelMax = 10, kCtlCount = 11;

// Times taken inside the single-workgroup solve, in ticks of the device's wall clock: its cycles, and the
// lattice sweeps in them, with their numbers.
constexpr int kClkIter = 0, kClkCycles = 1, kClkSmooth = 2, kClkPasses = 3, kClkCount = 4;

struct SmallArgs {
    GShape sh;
    double tol, margin;  // margin: what is aimed at, of the tolerance
    int maxit, fixed;    // fixed > 0: that many cycles, no test
    int step, history;   // step: the start is extrapolated in time from phi, prev, prev2
    double *prev, *prev2, *ctl;
    double* clock;       // adds to kClk*, or null
};
template <typename T>
void launch_small_solve(const Scalars& S, const Fields<T>& F, const GSub& G, const GTab& t, const SmallArgs& a,
                        hipStream_t st);

// A launched coarse grid in its own axes; the MGLevel beside it has its compact ones.
struct GTrans {
    int d[3];
    unsigned n;
    int lead, of[3], oc[3];
    double inv_nx, inv_ny;
};

// face coefficients of grid C (from the lattice, from grid Cf), residuals restricted to it with
// the start of its correction (red_omega > 0: with the first red pass), and its correction
// interpolated (onto the lattice, onto grid Cf)
template <typename T>
void launch_g_coarsen0(const Scalars& S, const Fields<T>& F, const GTrans& C, const MGLevel& M, const GTab& t,
                       hipStream_t st);
void launch_g_coarsen(const GTrans& Cf, const MGLevel& Mf, const GTrans& C, const MGLevel& M, const GTab& t,
                      hipStream_t st);
template <typename T>
void launch_g_restrict0(const Scalars& S, const Fields<T>& F, const GTrans& C, const MGLevel& M, const GTab& t,
                        double red_omega, hipStream_t st);
void launch_g_restrict(const GTrans& Cf, const MGLevel& Mf, const GTrans& C, const MGLevel& M, const GTab& t,
                       double red_omega, hipStream_t st);
template <typename T>
void launch_g_prolong0(const Scalars& S, const Fields<T>& F, const GTrans& C, const MGLevel& M, const GTab& t,
                       hipStream_t st);
void launch_g_prolong(const GTrans& Cf, const MGLevel& Mf, const GTrans& C, const MGLevel& M, const GTab& t,
                      hipStream_t st);
void launch_g_tail_build(const GSub& G, const GTab& t, const MGLevel& M, void* rows, hipStream_t st);
void launch_g_tail(const GSub& G, const GTab& t, const MGLevel& M, const void* rows, const GShape& sh, hipStream_t st);

}  // namespace ek
