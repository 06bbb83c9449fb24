// Device helpers of the lattice Poisson equation shared by the site-order kernels
// (ek_kernels.hip) and the column kernels (ek_columns.hip): the row, the relaxed update, the
// start of a coarse correction.
#pragma once

#include "ek_device.h"

namespace ek {

// Inside a multigrid solve the lattice potential and charge can be held colour-split (SP):
// the sites of colour (x + y + z) % 2 = 1 follow those of colour 0, each colour in site
// order, so a colour pass reads and writes whole cache lines of its own colour.  Axes are
// even there, site i of colour c sits at c N/2 + i/2, and every neighbour has the other
// colour.  The permittivity stays in site order.
template <bool SP>
__device__ __forceinline__ unsigned cidx(const Scalars& S, unsigned i, int color) {
    return SP ? (color ? (S.N >> 1) : 0u) + (i >> 1) : i;
}

// The sums of a row: twice the six face permittivities ((ei + ej), 0 for a face left out) and
// the potentials across them, without contraction, so that every kernel rounds a row the same
// way whatever surrounds it (the factor 1/2 moves no bits).  The two sides of an axis may be
// swapped: a mirrored lattice gives the mirrored row, and a kernel need not sort them.
__device__ __forceinline__ void poisson_sums(double xl, double xh, double yl, double yh, double zl, double zh, double pxa,
                                             double pxb, double pya, double pyb, double pza, double pzb, double& diag,
                                             double& offsum) {
#pragma clang fp contract(off)
    diag = 0.5 * (((xl + xh) + (yl + yh)) + (zl + zh));
    offsum = 0.5 * (((xl * pxa + xh * pxb) + (yl * pya + yh * pyb)) + (zl * pza + zh * pzb));
}
// The polarisation term: the sum over the faces of eps_f (E_ext . c_d).
__device__ __forceinline__ double poisson_polar(const Scalars& S, double xl, double xh, double yl, double yh, double zl,
                                                double zh) {
    return 0.5 * fma(S.E_ext[2], zh - zl, fma(S.E_ext[1], yh - yl, S.E_ext[0] * (xh - xl)));
}

// The row with the neighbour potentials supplied by pv(j, colour, ox, oy, oz) for the
// neighbour j at offset (ox, oy, oz); poisson_row reads them from F.phi.  Every
// operand is fetched before the arithmetic: the faces that an axis of length 1 or a wall
// leaves out are fetched too (their indices are lattice sites: the site itself, or a wall
// layer) and then not used, so the loads carry no branches and issue together.
// The permittivities come from ev(j, ox, oy, oz) the same way and the charge from qv()
// (poisson_row: from F.eps and F.q); mean is the source's mean (F.scal[0]).
template <typename T, bool SP, typename PV, typename EV, typename QV>
__device__ __forceinline__ void poisson_row_ve(unsigned i, int x, int y, int z, const Scalars& S, const Fields<T>& F,
                                               PV&& pv, EV&& ev, QV&& qv, double mean, double& diag, double& offsum,
                                               double& src) {
    const int own = SP ? ((x + y + z) & 1) : 0, nb = own ^ 1;
    const unsigned xa = i + (x == 0 ? S.nx - 1 : -1), xb = i + (x == S.nx - 1 ? -(S.nx - 1) : 1);
    const unsigned ya = i + (y == 0 ? (S.ny - 1) * S.nx : -S.nx), yb = i + (y == S.ny - 1 ? -(S.ny - 1) * S.nx : S.nx);
    const unsigned za = i + (z == 0 ? (S.nz - 1) * S.nxy : -S.nxy), zb = i + (z == S.nz - 1 ? -(S.nz - 1) * S.nxy : S.nxy);
    const double ei = ev(i, 0, 0, 0);
    const double exa = ev(xa, -1, 0, 0), exb = ev(xb, 1, 0, 0), eya = ev(ya, 0, -1, 0), eyb = ev(yb, 0, 1, 0),
                 eza = ev(za, 0, 0, -1), ezb = ev(zb, 0, 0, 1);
    const double pxa = pv(xa, nb, -1, 0, 0), pxb = pv(xb, nb, 1, 0, 0), pya = pv(ya, nb, 0, -1, 0),
                 pyb = pv(yb, nb, 0, 1, 0), pza = pv(za, nb, 0, 0, -1), pzb = pv(zb, nb, 0, 0, 1);
    double s = qv();
    // A face that is left out (an axis of length 1, a wall) is taken with a zero
    // coefficient: adding +0 leaves every sum as it is, and the row has no branches, so the
    // loads of consecutive rows can overlap.
    const bool onx = S.nx > 1, ony = S.ny > 1;
    const bool lo = S.nz > 1 && !(S.walls && z == S.z0), hi = S.nz > 1 && !(S.walls && z == S.z1);
    const double xl = onx ? ei + exa : 0.0, xh = onx ? ei + exb : 0.0;
    const double yl = ony ? ei + eya : 0.0, yh = ony ? ei + eyb : 0.0;
    const double zl = lo ? ei + eza : 0.0, zh = hi ? ei + ezb : 0.0;
    poisson_sums(xl, xh, yl, yh, zl, zh, pxa, pxb, pya, pyb, pza, pzb, diag, offsum);
    if (S.walls && z == S.z0) s += S.sigma0;
    if (S.walls && z == S.z1) s += S.sigma1;
    if (S.polar) s -= poisson_polar(S, xl, xh, yl, yh, zl, zh);
    src = s - mean;
}

// Over-relaxed Gauss-Seidel update of potential p, and the residual, of a row; one expression
// for every kernel (see poisson_sums).
__device__ __forceinline__ double sor_update(double p, double diag, double offsum, double src, double omega) {
    return fma(omega, (offsum + src) / diag - p, p);
}
__device__ __forceinline__ double row_residual(double p, double diag, double offsum, double src) {
    return fma(-diag, p, src + offsum);
}

__device__ __forceinline__ unsigned lid(const MGLevel& L, int x, int y, int z) {
    return (unsigned)x + (unsigned)L.nx * ((unsigned)y + (unsigned)L.ny * (unsigned)z);
}

// Start of a coarse grid's correction: zero, except that with red_omega > 0 the red cells
// ((I + J + K) even) take the first red pass of the pre-smoothing here.  From a zero
// correction every neighbour term of that pass vanishes and it reduces to
// omega s / diag, written as the sweep writes it (same operand order), so the grid's
// first separate pass can be skipped.
__device__ __forceinline__ void coarse_start(const MGLevel& C, int I, int J, int K, unsigned t, double s,
                                             double red_omega) {
    double v = 0.0;
    if (red_omega > 0.0 && ((I + J + K) & 1) == 0) {
        const int xm = wrapc(I - 1, C.nx), ym = wrapc(J - 1, C.ny), zm = wrapc(K - 1, C.nz);
        const double diag = C.ax[t] + C.ax[lid(C, xm, J, K)] + C.ay[t] + C.ay[lid(C, I, ym, K)] + C.az[t] +
                            C.az[lid(C, I, J, zm)];
        if (diag > 0.0) {
            const double p = 0.0, off = 0.0;
            v = p + red_omega * ((off + s) / diag - p);
        }
    }
    C.phi[t] = v;
}

// Interpolation of the coarse correction: along z between the own coarse cell and the
// neighbour towards the site, then the 3/4, 1/4 combination of x and of y.
__device__ __forceinline__ double prolong_z(double w0, double own, double w1, double nbr) {
    return fma(w1, nbr, w0 * own);
}
__device__ __forceinline__ double prolong_q(double own, double nbr) { return fma(0.25, nbr, 0.75 * own); }

}  // namespace ek
