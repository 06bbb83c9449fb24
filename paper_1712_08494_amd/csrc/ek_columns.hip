// Lattice passes of the Poisson solve that march up a column of planes (two colours, even axes).
//
// A thread owns one pair of sites (2 m, 2 m + 1) of a row and takes it through a chunk of planes.
// What the passes of one thread per site spent most of their instructions on is done once a
// column: the division of the site index into coordinates, the periodic neighbours in x and y.
// The plane is the same for a whole workgroup, so walls and the periodic neighbour in z are scalar.
// The pair's potential and permittivity of three planes stay in registers: the neighbours
// in z, and the one in x inside the pair, cost no load, and a row loads 10 values instead of 15.
// The rows are bound by HBM (19 B a lattice site and colour pass in FP32); measured per launch, one
// thread per site -> columns:
//                               256^3 FP32, spheres    128^3 FP64 (all include ~4 us of launch)
//   colour pass                  78 -> 62 us (5.1 TB/s)    13.0 -> 11.9
//   black pass from blk          94 -> 75                  12.7 -> 12.0
//   residual sums (mean of two) 166 -> 113                 27.7 -> 19.4
//   restriction                 118 -> 87                  20.3 -> 14.3
//   interpolation + red pass    148 -> 93                  21.3 -> 15.7
// At 32^3 every pass is launch and latency (6 to 9 us both ways).
#include <algorithm>

#include "ek_poisson.h"

namespace ek {

template <typename T> struct PairOf;
template <> struct PairOf<float> { using type = float2; };
template <> struct PairOf<double> { using type = double2; };

// Planes per thread: as many as leave `waves` waves on the chip.
static int column_planes(unsigned cells, int planes, unsigned waves) {
    const unsigned per_plane = (cells + 63) / 64;
    return std::max(1, std::min(16, (int)((unsigned long long)per_plane * (unsigned)planes / waves)));
}

// Waves wanted of a pass, four per SIMD where a thread owns a pair and two where it owns the
// columns of a coarse cell.  From 1024 to 8192 (8 planes to 1 at 128^3): sweep 14.4 to 11.8 us, level
// from 4096; restriction 13.0 us at 2048 and 13.7 above; at 256^3 all are within 5 %.
constexpr unsigned kSiteWaves = 4096, kCellWaves = 2048;

struct ColumnGrid {
    unsigned tiles;  // workgroups per chunk of planes
    int planes;      // planes per chunk
    unsigned blocks;
};
static ColumnGrid column_grid(unsigned cells, int planes, unsigned waves) {
    ColumnGrid g;
    g.tiles = (cells + kBlock - 1) / kBlock;
    g.planes = column_planes(cells, planes, waves);
    const unsigned chunks = (unsigned)((planes + g.planes - 1) / g.planes);
    g.blocks = (g.tiles * chunks + 7) / 8 * 8;
    return g;
}

// Chunk and tile of a workgroup: XCD k takes a contiguous range of both (see xcd_linear).
__device__ __forceinline__ void column_place(unsigned tiles, unsigned& chunk, unsigned& tile) {
    const unsigned nb = gridDim.x, b = blockIdx.x;
    const unsigned lb = (b & 7u) * (nb >> 3) + (b >> 3);
    chunk = lb / tiles;
    tile = lb - chunk * tiles;
}

// A thread's pair: c = m + (nx / 2) y within its plane, and the offsets to the pairs next to it.
struct Pairs {
    unsigned c;
    int y, xl, xh, ya, yb;
};
__device__ __forceinline__ Pairs pair_at(const Scalars& S, unsigned c) {
    const unsigned hx = (unsigned)S.nx >> 1;
    Pairs P;
    P.c = c;
    P.y = (int)div_exact(c, S.inv_hx);
    const unsigned m = c - (unsigned)P.y * hx;
    P.xl = m == 0 ? (int)hx - 1 : -1;
    P.xh = m == hx - 1 ? 1 - (int)hx : 1;
    P.ya = P.y == 0 ? (S.ny - 1) * (int)hx : -(int)hx;
    P.yb = P.y == S.ny - 1 ? -(S.ny - 1) * (int)hx : (int)hx;
    return P;
}

// The row of one site of a pair: po, eo the neighbour in x outside the pair, ps, es the one inside;
// p the site's parity in x.
__device__ __forceinline__ void column_row(const Scalars& S, int z, int p, double ei, double es, double eo, double eya,
                                           double eyb, double eza, double ezb, double ps, double po, double pya,
                                           double pyb, double pza, double pzb, double q, double mean, double& diag,
                                           double& offsum, double& src) {
    const double xs = ei + es, xo = ei + eo, yl = ei + eya, yh = ei + eyb;
    double zl = ei + eza, zh = ei + ezb, s = q;
    if (S.walls) {
        if (z == S.z0) zl = 0.0;
        if (z == S.z1) zh = 0.0;
    }
    poisson_sums(xs, xo, yl, yh, zl, zh, ps, po, pya, pyb, pza, pzb, diag, offsum);
    if (S.walls && z == S.z0) s += S.sigma0;
    if (S.walls && z == S.z1) s += S.sigma1;
    if (S.polar) s -= poisson_polar(S, p ? xs : xo, p ? xo : xs, yl, yh, zl, zh);
    src = s - mean;
}

// One colour of a sweep: own holds the colour's potentials (updated), oth the other colour's; cur
// the values to relax from (own, or the black values the interpolation left apart).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_sor_col(Scalars S, int color, double omega, const T* __restrict__ eps,
                                                    const T* __restrict__ q, const double* __restrict__ oth,
                                                    const double* cur, double* own, const double* __restrict__ scal,
                                                    int zc, unsigned tiles) {
    using P2 = typename PairOf<T>::type;
    unsigned chunk, tile;
    column_place(tiles, chunk, tile);
    const int za = S.z0 + (int)chunk * zc, zb = min(za + zc - 1, S.z1);
    const unsigned hxy = (unsigned)S.nxy >> 1, c = tile * kBlock + threadIdx.x;
    if (za > S.z1 || c >= hxy) return;
    const Pairs P = pair_at(S, c);
    const double mean = scal[0];
    auto plane = [&](int z) { return hxy * (unsigned)(z < 0 ? S.nz - 1 : (z >= S.nz ? 0 : z)); };
    auto pair = [&](unsigned h) { return *reinterpret_cast<const P2*>(eps + 2 * (size_t)h); };
    const unsigned hm = plane(za - 1) + c, h0 = plane(za) + c;
    double pm = oth[hm], pc = oth[h0];
    P2 em = pair(hm), ec = pair(h0);
    int p = (color + P.y + za) & 1;
    for (int z = za; z <= zb; ++z, p ^= 1) {
        const unsigned h = plane(z) + c, hp = plane(z + 1) + c;
        const double pp = oth[hp];
        const P2 ep = pair(hp);
        const unsigned ho = h + (unsigned)(p ? P.xh : P.xl);
        const double po = oth[ho], pya = oth[h + (unsigned)P.ya], pyb = oth[h + (unsigned)P.yb];
        const T eo = eps[2 * (size_t)ho + (p ^ 1)], eya = eps[2 * (size_t)(h + (unsigned)P.ya) + p],
                eyb = eps[2 * (size_t)(h + (unsigned)P.yb) + p];
        const double v = cur[h];
        double diag, offsum, src;
        column_row(S, z, p, (double)(p ? ec.y : ec.x), (double)(p ? ec.x : ec.y), (double)eo, (double)eya, (double)eyb,
                   (double)(p ? em.y : em.x), (double)(p ? ep.y : ep.x), pc, po, pya, pyb, pm, pp, (double)q[h], mean,
                   diag, offsum, src);
        own[h] = diag > 0.0 ? sor_update(v, diag, offsum, src, omega) : v;  // an isolated site keeps its value
        pm = pc;
        pc = pp;
        em = ec;
        ec = ep;
    }
}

template <typename T>
void launch_sor_col(const Scalars& S, const Fields<T>& F, int color, double omega, const double* cur, hipStream_t st) {
    const unsigned hxy = (unsigned)S.nxy / 2, half = S.N / 2;
    const ColumnGrid g = column_grid(hxy, S.z1 - S.z0 + 1, kSiteWaves);
    double* own = F.phi + (color ? half : 0u);
    hipLaunchKernelGGL(k_sor_col<T>, dim3(g.blocks), dim3(kBlock), 0, st, S, color, omega, F.eps,
                       F.q + (color ? half : 0u), F.phi + (color ? 0u : half), cur ? cur : own, own, F.scal, g.planes,
                       g.tiles);
}

// Residual sums (see residual_body), pair by pair up the column.
// SP: colour-split fields; otherwise site order, and the colour-split copies (phis, qs non-null)
// are written on the way, wall layers included.
template <typename T, bool SP>
__global__ __launch_bounds__(kBlock) void k_residual_col(Scalars S, Fields<T> F, double* __restrict__ phis,
                                                         T* __restrict__ qs, int zc, unsigned tiles) {
    using P2 = typename PairOf<T>::type;
    unsigned chunk, tile;
    column_place(tiles, chunk, tile);
    const int za = (int)chunk * zc, zb = min(za + zc, S.nz) - 1;
    const unsigned hxy = (unsigned)S.nxy >> 1, half = S.N >> 1, c = tile * kBlock + threadIdx.x;
    double acc[3] = {0.0, 0.0, 0.0};
    if (za < S.nz && c < hxy) {
        const Pairs P = pair_at(S, c);
        const double mean = F.scal[0];
        const double* __restrict__ phi = F.phi;
        const T *__restrict__ eps = F.eps, *__restrict__ q = F.q;
        auto plane = [&](int z) { return hxy * (unsigned)(z < 0 ? S.nz - 1 : (z >= S.nz ? 0 : z)); };
        // the potentials of the pair at h by site, w the x parity of its colour-0 site
        auto pot = [&](unsigned h, int w) {
            if (!SP) return *reinterpret_cast<const double2*>(phi + 2 * (size_t)h);
            const double a = phi[h], b = phi[half + h];
            return w ? double2{b, a} : double2{a, b};
        };
        auto one = [&](unsigned h, int col, int x) { return SP ? phi[(col ? half : 0u) + h] : phi[2 * (size_t)h + x]; };
        auto pair = [&](unsigned h) { return *reinterpret_cast<const P2*>(eps + 2 * (size_t)h); };
        const unsigned hm = plane(za - 1) + c, h0 = plane(za) + c;
        int w = (P.y + za) & 1;
        double2 pm = pot(hm, w ^ 1), pc = pot(h0, w);
        P2 em = pair(hm), ec = pair(h0);
        for (int z = za; z <= zb; ++z, w ^= 1) {
            const unsigned h = plane(z) + c, hp = plane(z + 1) + c;
            const double2 pp = pot(hp, w ^ 1);
            const P2 ep = pair(hp);
            const unsigned hl = h + (unsigned)P.xl, hh = h + (unsigned)P.xh, ha = h + (unsigned)P.ya,
                           hb = h + (unsigned)P.yb;
            const double pl = one(hl, w ^ 1, 1), ph = one(hh, w, 0);  // sites 2 m - 1 and 2 m + 2
            const T el = eps[2 * (size_t)hl + 1], eh = eps[2 * (size_t)hh];
            const double2 pya = pot(ha, w ^ 1), pyb = pot(hb, w ^ 1);
            const P2 eya = pair(ha), eyb = pair(hb);
            T q0, q1;  // of the sites 2 m and 2 m + 1
            if (SP) {
                const T a = q[h], b = q[half + h];
                q0 = w ? b : a;
                q1 = w ? a : b;
            } else {
                const P2 v = *reinterpret_cast<const P2*>(q + 2 * (size_t)h);
                q0 = v.x;
                q1 = v.y;
            }
            if (!SP && phis) {
                phis[h] = w ? pc.y : pc.x;
                phis[half + h] = w ? pc.x : pc.y;
                qs[h] = w ? q1 : q0;
                qs[half + h] = w ? q0 : q1;
            }
            double diag, off, src0, src1;
            column_row(S, z, 0, (double)ec.x, (double)ec.y, (double)el, (double)eya.x, (double)eyb.x, (double)em.x,
                       (double)ep.x, pc.y, pl, pya.x, pyb.x, pm.x, pp.x, (double)q0, mean, diag, off, src0);
            const double r0 = row_residual(pc.x, diag, off, src0);
            column_row(S, z, 1, (double)ec.y, (double)ec.x, (double)eh, (double)eya.y, (double)eyb.y, (double)em.y,
                       (double)ep.y, pc.x, ph, pya.y, pyb.y, pm.y, pp.y, (double)q1, mean, diag, off, src1);
            const double r1 = row_residual(pc.y, diag, off, src1);
            if (z >= S.z0 && z <= S.z1) {
                acc[0] += r0 * r0 + r1 * r1;
                acc[1] += src0 * src0 + src1 * src1;
                acc[2] += pc.x + pc.y;
            }
            pm = pc;
            pc = pp;
            em = ec;
            ec = ep;
        }
    }
    const bool mx[3] = {false, false, false};
    block_reduce_store<3>(acc, mx, F.red, blockIdx.x, gridDim.x);
}

// (the sums go to three records of the reduction scratch per workgroup: at most as many as
// site_blocks)
static ColumnGrid residual_grid(const Scalars& S) {
    ColumnGrid g = column_grid((unsigned)S.nxy / 2, S.nz, kSiteWaves);
    const unsigned most = site_blocks(S.N);
    if (g.blocks > most) {
        const unsigned chunks = std::max(1u, most / g.tiles);
        g.planes = (int)(((unsigned)S.nz + chunks - 1) / chunks);
        g.blocks = most;
    }
    return g;
}

// Even axes, and a plane of a wave of pairs at least: a 2 x 2 x 2500 column would leave two threads of
// a workgroup with 60 planes each.
bool columns_fit(const Scalars& S) { return S.nx % 2 == 0 && S.ny % 2 == 0 && S.nz % 2 == 0 && S.nxy >= 128; }
unsigned residual_col_blocks(const Scalars& S) { return residual_grid(S).blocks; }

template <typename T>
void launch_residual_col(const Scalars& S, const Fields<T>& F, bool split, double* phis, T* qs, hipStream_t st) {
    const ColumnGrid g = residual_grid(S);
    if (split)
        hipLaunchKernelGGL((k_residual_col<T, true>), dim3(g.blocks), dim3(kBlock), 0, st, S, F, (double*)nullptr,
                           (T*)nullptr, g.planes, g.tiles);
    else
        hipLaunchKernelGGL((k_residual_col<T, false>), dim3(g.blocks), dim3(kBlock), 0, st, S, F, phis, qs, g.planes,
                           g.tiles);
}

// Residuals of the lattice summed over the children of each cell of the first coarse grid, with the
// start of its correction (the sums and their order are those of restrict_fine_body).  A thread owns
// the columns of a coarse cell: two rows of a pair, two planes a cell.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_restrict_col(Scalars S, Fields<T> F, MGLevel C, double red_omega, int zc,
                                                         unsigned tiles) {
    using P2 = typename PairOf<T>::type;
    unsigned chunk, tile;
    column_place(tiles, chunk, tile);
    const int Ka = (int)chunk * zc, Kb = min(Ka + zc, C.nz) - 1;
    const unsigned hx = (unsigned)C.nx, hxy = (unsigned)S.nxy >> 1, half = S.N >> 1;
    const unsigned c = tile * kBlock + threadIdx.x;
    if (Ka >= C.nz || c >= hx * (unsigned)C.ny) return;
    const int J = (int)div_exact(c, S.inv_hx), I = (int)(c - (unsigned)J * hx);
    const Pairs P = pair_at(S, c + hx * (unsigned)J);  // row 2 J
    const int yb = 2 * J + 1 == S.ny - 1 ? -(S.ny - 1) * (int)hx : (int)hx;
    const double mean = F.scal[0];
    const double* __restrict__ phi = F.phi;
    const T *__restrict__ eps = F.eps, *__restrict__ q = F.q;
    auto plane = [&](int z) { return hxy * (unsigned)(z < 0 ? S.nz - 1 : (z >= S.nz ? 0 : z)); };
    auto pot = [&](unsigned h, int w) {
        const double a = phi[h], b = phi[half + h];
        return w ? double2{b, a} : double2{a, b};
    };
    auto pair = [&](unsigned h) { return *reinterpret_cast<const P2*>(eps + 2 * (size_t)h); };
    // [plane][row]: planes 2 K - 1 .. 2 K + 2 of the cell; in row r of plane z the colour-0 site has the
    // x parity w = (r + z) & 1
    double2 v[4][2];
    P2 e[4][2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const unsigned h = plane(2 * Ka - 1 + k) + P.c + r * hx;
            v[k][r] = pot(h, (r + k + 1) & 1);
            e[k][r] = pair(h);
        }
    for (int K = Ka; K <= Kb; ++K) {
        // every operand of the cell's eight rows first, so that their loads overlap
        double2 vo[2][2];  // rows 2 J - 1, 2 J + 2
        P2 eo[2][2];
        double vl[2][2], vh[2][2];  // sites 2 I - 1, 2 I + 2
        T el[2][2], eh[2][2], q0[2][2], q1[2][2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const unsigned h = plane(2 * K + k) + P.c, hp = plane(2 * K + k + 1) + P.c;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int w = (r + k) & 1;
                const unsigned hr = h + r * hx, hl = hr + (unsigned)P.xl, hh = hr + (unsigned)P.xh,
                               ho = hr + (unsigned)(r ? yb : P.ya);
                v[k + 2][r] = pot(hp + r * hx, w ^ 1);
                e[k + 2][r] = pair(hp + r * hx);
                vo[k][r] = pot(ho, w ^ 1);
                eo[k][r] = pair(ho);
                vl[k][r] = phi[(w ? 0u : half) + hl];
                vh[k][r] = phi[(w ? half : 0u) + hh];
                el[k][r] = eps[2 * (size_t)hl + 1];
                eh[k][r] = eps[2 * (size_t)hh];
                const T qa = q[hr], qb = q[half + hr];
                q0[k][r] = w ? qb : qa;
                q1[k][r] = w ? qa : qb;
            }
        }
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int z = 2 * K + k;
            const double2(&m)[2] = v[k], (&o)[2] = v[k + 1], (&p)[2] = v[k + 2];
            const P2(&em)[2] = e[k], (&ec)[2] = e[k + 1], (&ep)[2] = e[k + 2];
            double res[2][2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const double2 ya = r ? o[0] : vo[k][0], yh = r ? vo[k][1] : o[1];
                const P2 eya = r ? ec[0] : eo[k][0], eyb = r ? eo[k][1] : ec[1];
                double diag, off, src;
                column_row(S, z, 0, (double)ec[r].x, (double)ec[r].y, (double)el[k][r], (double)eya.x, (double)eyb.x,
                           (double)em[r].x, (double)ep[r].x, o[r].y, vl[k][r], ya.x, yh.x, m[r].x, p[r].x,
                           (double)q0[k][r], mean, diag, off, src);
                res[r][0] = row_residual(o[r].x, diag, off, src);
                column_row(S, z, 1, (double)ec[r].y, (double)ec[r].x, (double)eh[k][r], (double)eya.y, (double)eyb.y,
                           (double)em[r].y, (double)ep[r].y, o[r].x, vh[k][r], ya.y, yh.y, m[r].y, p[r].y,
                           (double)q1[k][r], mean, diag, off, src);
                res[r][1] = row_residual(o[r].y, diag, off, src);
            }
            if (z >= S.z0 && z <= S.z1) sum += (res[0][0] + res[0][1]) + (res[1][0] + res[1][1]);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                v[k][r] = v[k + 2][r];
                e[k][r] = e[k + 2][r];
            }
        const unsigned t = lid(C, I, J, K);
        C.s[t] = sum;
        coarse_start(C, I, J, K, t, sum, red_omega);
    }
}

template <typename T>
void launch_restrict_col(const Scalars& S, const Fields<T>& F, const MGLevel& C, double red_omega, hipStream_t st) {
    const ColumnGrid g = column_grid((unsigned)C.nx * (unsigned)C.ny, C.nz, kCellWaves);
    hipLaunchKernelGGL(k_restrict_col<T>, dim3(g.blocks), dim3(kBlock), 0, st, S, F, C, red_omega, g.planes, g.tiles);
}

// The interpolation from the first coarse grid with the first red pass of the post-smoothing.  A
// thread owns the columns of a coarse cell.  At each plane its two red sites are updated from the
// interpolated values of the two black sites of the 2 x 2 block (the plane's own, the one before and
// the one after: computed once, kept) and of the four black sites beside it.  The block's
// interpolated black values go to blk, from which the black pass relaxes: in place they could
// reach a neighbouring thread that still needs the old values.  Of the coarse potential the 3 x 3
// cells around the thread's column in three planes are in registers; each lattice plane takes their
// combination along z once, then that along x and y per site (prolong_corr's expression).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_prolong_red_col(Scalars S, Fields<T> F, MGLevel C, double omega,
                                                            double* __restrict__ blk, int zc, unsigned tiles) {
    using P2 = typename PairOf<T>::type;
    unsigned chunk, tile;
    column_place(tiles, chunk, tile);
    const int Ka = (int)chunk * zc, Kb = min(Ka + zc, C.nz) - 1;
    const unsigned hx = (unsigned)C.nx, hxy = (unsigned)S.nxy >> 1, half = S.N >> 1;
    const unsigned c = tile * kBlock + threadIdx.x, cells = hx * (unsigned)C.ny;
    if (Ka >= C.nz || c >= cells) return;
    const int J = (int)div_exact(c, S.inv_hx);
    const Pairs P = pair_at(S, c + hx * (unsigned)J);  // row 2 J
    const int yb = 2 * J + 1 == S.ny - 1 ? -(S.ny - 1) * (int)hx : (int)hx;
    const double mean = F.scal[0];
    double* __restrict__ red = F.phi;
    const double* __restrict__ black = F.phi + half;
    const double* __restrict__ cphi = C.phi;
    const T *__restrict__ eps = F.eps, *__restrict__ q = F.q;
    auto plane = [&](int z) { return hxy * (unsigned)(z < 0 ? S.nz - 1 : (z >= S.nz ? 0 : z)); };
    auto pair = [&](unsigned h) { return *reinterpret_cast<const P2*>(eps + 2 * (size_t)h); };
    int co[3][3];
    {
        const int ya = J == 0 ? (C.ny - 1) * (int)hx : -(int)hx, yu = J == C.ny - 1 ? -(C.ny - 1) * (int)hx : (int)hx;
#pragma unroll
        for (int oy = 0; oy < 3; ++oy)
#pragma unroll
            for (int ox = 0; ox < 3; ++ox)
                co[oy][ox] = (int)c + (oy == 0 ? ya : (oy == 2 ? yu : 0)) + (ox == 0 ? P.xl : (ox == 2 ? P.xh : 0));
    }
    using Cells = double[3][3];
    auto coarse = [&](int K, Cells& V) {
        const double* p = cphi + (size_t)cells * (unsigned)wrapc(K, C.nz);
#pragma unroll
        for (int oy = 0; oy < 3; ++oy)
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) V[oy][ox] = p[co[oy][ox]];
    };
    // the combination along z at plane z: own cell K, neighbour Kn (not wrapped)
    auto along_z = [&](int K, int Kn, const Cells& own, const Cells& nbr, Cells& Z) {
        const int Kw = wrapc(K, C.nz), d = Kn - K;
        const double wz = S.walls && (Kw + d < 0 || Kw + d >= C.nz) ? 0.0 : 0.25;
#pragma unroll
        for (int oy = 0; oy < 3; ++oy)
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) Z[oy][ox] = prolong_z(1.0 - wz, own[oy][ox], wz, nbr[oy][ox]);
    };
    // correction of the site (2 I + rx, 2 J + ry) from a plane's combination, rx, ry in -1 .. 2
    auto corr = [&](const Cells& Z, int rx, int ry) {
        const int ox = 1 + (rx >> 1), oy = 1 + (ry >> 1), nx = (rx & 1) ? ox + 1 : ox - 1,
                  ny = (ry & 1) ? oy + 1 : oy - 1;
        return prolong_q(prolong_q(Z[oy][ox], Z[oy][nx]), prolong_q(Z[ny][ox], Z[ny][nx]));
    };
    Cells A, B, D, Z;  // coarse planes K - 1, K, K + 1; the combination of the plane at hand
    coarse(Ka - 1, A);
    coarse(Ka, B);
    // black values of the block at the plane before and the one at hand: [r] in row 2 J + r
    double bm[2], bc[2];
    P2 em[2], ec[2];
    {
        const unsigned hm = plane(2 * Ka - 1) + P.c, h0 = plane(2 * Ka) + P.c;
        along_z(Ka - 1, Ka, A, B, Z);  // an odd plane: black at (0, 0) and (1, 1)
        bm[0] = black[hm] + corr(Z, 0, 0);
        bm[1] = black[hm + hx] + corr(Z, 1, 1);
        along_z(Ka, Ka - 1, B, A, Z);  // an even plane: black at (1, 0) and (0, 1)
        bc[0] = black[h0] + corr(Z, 1, 0);
        bc[1] = black[h0 + hx] + corr(Z, 0, 1);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            em[r] = pair(hm + r * hx);
            ec[r] = pair(h0 + r * hx);
        }
    }
    for (int K = Ka; K <= Kb; ++K) {
        coarse(K + 1, D);
#pragma unroll
        for (int cz = 0; cz < 2; ++cz) {
            const int z = 2 * K + cz;
            const unsigned h = plane(z) + P.c, hp = plane(z + 1) + P.c;
            P2 ep[2];
            double own[2], px[2], py[2];  // by row: red value, black neighbours outside the block
            T ex[2], ey[2], qr[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int x = r ^ cz;  // the red site's parity in x
                const unsigned hr = h + r * hx, hox = hr + (unsigned)(x ? P.xh : P.xl),
                               hoy = hr + (unsigned)(r ? yb : P.ya);
                ep[r] = pair(hp + r * hx);
                own[r] = red[hr] + corr(Z, x, r);
                px[r] = black[hox] + corr(Z, x ? 2 : -1, r);
                py[r] = black[hoy] + corr(Z, x, r ? 2 : -1);
                ex[r] = eps[2 * (size_t)hox + (x ^ 1)];
                ey[r] = eps[2 * (size_t)hoy + x];
                qr[r] = q[hr];
            }
            if (cz == 0)
                along_z(K, K + 1, B, D, Z);
            else
                along_z(K + 1, K, D, B, Z);
            double bp[2];  // black at the plane after, above the red sites
            bp[0] = black[hp] + corr(Z, cz, 0);
            bp[1] = black[hp + hx] + corr(Z, cz ^ 1, 1);
            const bool in = z >= S.z0 && z <= S.z1;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int x = r ^ cz;
                auto at = [&](const P2& e, int k) { return (double)(k ? e.y : e.x); };
                const double ei = at(ec[r], x), ein = at(ec[r ^ 1], x), eout = (double)ey[r];
                double diag, off, src;
                column_row(S, z, x, ei, at(ec[r], x ^ 1), (double)ex[r], r ? ein : eout, r ? eout : ein, at(em[r], x),
                           at(ep[r], x), bc[r], px[r], r ? bc[0] : py[0], r ? py[1] : bc[1], bm[r], bp[r], (double)qr[r],
                           mean, diag, off, src);
                if (in) {
                    red[h + r * hx] = diag > 0.0 ? sor_update(own[r], diag, off, src, omega) : own[r];
                    blk[h + r * hx] = bc[r];
                }
            }
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                bm[r] = bc[r];
                bc[r] = bp[r];
                em[r] = ec[r];
                ec[r] = ep[r];
            }
        }
#pragma unroll
        for (int oy = 0; oy < 3; ++oy)
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) B[oy][ox] = D[oy][ox];
    }
}

template <typename T>
void launch_prolong_red_col(const Scalars& S, const Fields<T>& F, const MGLevel& C, double omega, double* blk,
                            hipStream_t st) {
    const ColumnGrid g = column_grid((unsigned)C.nx * (unsigned)C.ny, C.nz, kCellWaves);
    hipLaunchKernelGGL(k_prolong_red_col<T>, dim3(g.blocks), dim3(kBlock), 0, st, S, F, C, omega, blk, g.planes,
                       g.tiles);
}

#define EK_COL_INST(T)                                                                                             \
    template void launch_sor_col<T>(const Scalars&, const Fields<T>&, int, double, const double*, hipStream_t);    \
    template void launch_residual_col<T>(const Scalars&, const Fields<T>&, bool, double*, T*, hipStream_t);        \
    template void launch_restrict_col<T>(const Scalars&, const Fields<T>&, const MGLevel&, double, hipStream_t);   \
    template void launch_prolong_red_col<T>(const Scalars&, const Fields<T>&, const MGLevel&, double, double*,      \
                                            hipStream_t);
EK_COL_INST(float)
EK_COL_INST(double)

}  // namespace ek
