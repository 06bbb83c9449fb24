// Multigrid for lattices of any size and for lattices small enough for one workgroup.
//
// The V-cycle of ek_kernels.hip halves every axis of lattices whose axes divide by 4 and
// stops where one no longer does.  The hierarchy here coarsens each axis by itself down to
// a few cells (GHier, built by gmg_hierarchy): runs of two cells, and one or two runs of three
// or a run of one where the length asks for it, so that every coarse axis has an even
// number of cells or one.  A box with odd sides, sides not divisible by 4, or one side far
// shorter than the others then has a full hierarchy with red-black colours on every coarse
// grid.  The operator is the same finite-volume one (Sec. II D): a coarse face coefficient is
// the sum of the fine faces it covers, scaled by the ratio of the distances between cell
// centres; residuals are summed over children; corrections are interpolated linearly per
// axis between cell centres, falling back to the parent at a wall.
//
// Two users:
//   - k_small_solve: the whole solve in one workgroup (time extrapolation of the start, the
//     V-cycles with the convergence test, gauge and wall layers) where the lattice fits LDS;
//   - launched lattice and upper grids (k_g_*), with the grids below in one workgroup
//     (k_g_tail).
// All sums run in a fixed order, so results are deterministic.
#include "ek_device.h"
#include "ek_gmg.h"

#include <algorithm>
#include <cmath>

namespace ek {

// ------------------------------------------------------------------------------------
// Hierarchy (host)
// ------------------------------------------------------------------------------------
namespace {

// Cells of an axis of n cells after coarsening, and the start of each: even, or one.
std::vector<int> axis_starts(int n) {
    std::vector<int> s;
    if (n <= 3) {
        s = {0, n};
        return s;
    }
    const int r = n & 3;
    const int nc = r == 0 ? n / 2 : (r == 1 ? (n - 1) / 2 : (r == 2 ? n / 2 - 1 : (n + 1) / 2));
    const int threes = r == 1 ? 1 : (r == 2 ? 2 : 0);  // at the end; r == 3 ends in a single cell
    int x = 0;
    for (int I = 0; I < nc; ++I) {
        s.push_back(x);
        x += I >= nc - threes ? 3 : 2;
    }
    s.push_back(n);
    return s;
}

}  // namespace

void gmg_hierarchy(const int (&dims)[3], const bool (&periodic)[3], GHier& H) {
    H = GHier{};
    int n[3] = {dims[0], dims[1], dims[2]};
    std::vector<double> edge[3];  // cell edges of the current grid, in lattice units
    for (int k = 0; k < 3; ++k)
        for (int x = 0; x <= n[k]; ++x) edge[k].push_back(x);
    // (a lattice of 9 to kDirect sites has one coarse grid: by its sweeps alone a ring of 32 sites took
    // 71 cycles a step and left 8.2e-11 of phi at a residual of 1e-10)
    auto more = [&]() {
        const long long sites = (long long)n[0] * n[1] * n[2];
        return sites > kDirect || (H.levels.empty() && sites > 8);
    };
    while (more() && (int)H.levels.size() < kGMaxLevels) {
        GLevelDesc D{};
        std::vector<double> ne[3];
        for (int k = 0; k < 3; ++k) {
            const std::vector<int> st = axis_starts(n[k]);
            const int nc = (int)st.size() - 1;
            const double L = edge[k].back();
            for (int b : st) ne[k].push_back(edge[k][b]);
            auto fc = [&](int x) { return 0.5 * (edge[k][x] + edge[k][x + 1]); };
            auto cc = [&](int I) { return 0.5 * (ne[k][I] + ne[k][I + 1]); };
            D.of[k] = (int)H.pn.size();
            D.oc[k] = (int)H.first.size();
            for (int I = 0; I < nc; ++I) {
                for (int x = st[I]; x < st[I + 1]; ++x) {
                    const double d = fc(x) - cc(I);
                    int nb = I;
                    double w = 0.0;
                    if (nc > 1 && d != 0.0) {
                        nb = I + (d > 0 ? 1 : -1);
                        double dist;
                        if (nb < 0 || nb >= nc) {
                            if (periodic[k]) {
                                nb = nb < 0 ? nc - 1 : 0;
                                dist = L - cc(nc - 1) + cc(0);
                            } else {
                                nb = I;
                                dist = 0.0;
                            }
                        } else {
                            dist = std::fabs(cc(nb) - cc(I));
                        }
                        w = dist > 0.0 ? std::fabs(d) / dist : 0.0;
                    }
                    H.pn.push_back((uint32_t)I | ((uint32_t)nb << 16));
                    H.w.push_back((float)w);
                }
                // the face towards I + 1: fine over coarse distance between the cell centres
                double ratio = 0.0;
                const int xl = st[I + 1] - 1;
                if (nc > 1 && (I + 1 < nc || periodic[k])) {
                    const double df = I + 1 < nc ? fc(xl + 1) - fc(xl) : L - fc(xl) + fc(0);
                    const double dc = I + 1 < nc ? cc(I + 1) - cc(I) : L - cc(I) + cc(0);
                    ratio = df / dc;
                }
                H.first.push_back(st[I]);
                H.ratio.push_back((float)ratio);
            }
            H.first.push_back(n[k]);
            H.ratio.push_back(0.0f);
            n[k] = nc;
            edge[k] = ne[k];
        }
        for (int k = 0; k < 3; ++k) D.d[k] = n[k];
        D.n = (unsigned)n[0] * (unsigned)n[1] * (unsigned)n[2];
        D.lead = n[0] > 1 ? 0 : (n[1] > 1 ? 1 : 2);
        H.levels.push_back(D);
    }
}

// Grids first .. last of a hierarchy as a workgroup holds them in LDS, with the axis tables
// between them (from_lattice: also those from the lattice to the first of them).
GSub gmg_sub(const GHier& H, int first, bool from_lattice) {
    GSub G{};
    const int nl = (int)H.levels.size(), t0 = from_lattice ? first : first + 1;
    G.pn0 = t0 < nl ? H.levels[t0].of[0] : (int)H.pn.size();
    G.first0 = t0 < nl ? H.levels[t0].oc[0] : (int)H.first.size();
    int off = 0;
    for (int l = first; l < nl; ++l) {
        const GLevelDesc& D = H.levels[l];
        GLds& L = G.L[G.nl++];
        const int e[3] = {D.d[D.lead], D.lead < 2 ? D.d[D.lead + 1] : 1, D.lead < 1 ? D.d[2] : 1};
        L.nx = D.d[0], L.ny = D.d[1], L.nz = D.d[2];
        L.ex = e[0], L.ey = e[1], L.ez = e[2];
        L.n = (int)D.n;
        L.lead = D.lead;
        L.off = off;
        L.inv_hx = e[0] >= 2 ? 1.0f / (e[0] / 2) : 1.0f;
        L.inv_ey = 1.0f / e[1];
        L.inv_nx = 1.0f / D.d[0];
        L.inv_ny = 1.0f / D.d[1];
        for (int k = 0; k < 3; ++k) {
            L.of[k] = l >= t0 ? D.of[k] - G.pn0 : 0;
            L.oc[k] = l >= t0 ? D.oc[k] - G.first0 : 0;
        }
        off += L.n;
    }
    G.cells = off;
    G.npn = (int)H.pn.size() - G.pn0;
    G.nfirst = (int)H.first.size() - G.first0;
    return G;
}

// LDS of a workgroup holding the grids of G: per cell the correction and right-hand side
// (FP64) and the row (neighbours and FP32 coefficients, 48 bytes), the axis tables, the
// inverse of the coarsest grid, and scratch residuals.
static size_t sub_bytes(const GSub& G, size_t scratch_cells) {
    const size_t tabs = ((size_t)G.npn * 8 + (size_t)G.nfirst * 4 + 15) & ~(size_t)15;
    return (size_t)G.cells * 64 + kDirect * kDirect * 8 + 64 * 8 + std::max((scratch_cells + 1) & ~(size_t)1, (size_t)(kDirect * kDirect)) * 8 + tabs + 32;
}

static size_t tail_bytes(const GSub& G) { return sub_bytes(G, G.nl ? (size_t)G.L[0].n : 0); }

// The first grid of the hierarchy from which on all of them fit one workgroup; -1: none.
int gmg_tail_first(const GHier& H) {
    const int nl = (int)H.levels.size();
    if (nl == 0 || H.levels[nl - 1].n > (unsigned)kDirect) return -1;
    int l = nl - 1;
    while (l > 0 && (long long)H.levels[l - 1].n * 64 <= (long long)kGmgLds &&
           tail_bytes(gmg_sub(H, l - 1, false)) <= kGmgLds)
        --l;
    return l;
}

bool gmg_small_fits(const GSub& G, unsigned ndomain) {
    return ndomain <= kSmallMost && sub_bytes(G, ndomain) + (size_t)ndomain * 8 <= kGmgLds;
}

// ------------------------------------------------------------------------------------
// Device: the grids in LDS
// ------------------------------------------------------------------------------------
// floor(a / d) for a, d below 2^20 from a rounded 1/d: (a + 1/2)/d stays 1/(2d) clear of an
// integer, more than the two FP32 roundings can move it.
__device__ __forceinline__ int fdiv(int a, float inv) { return (int)(((float)a + 0.5f) * inv); }

// The rows of a grid are kept in colour order (cell i of colour c at c n/2 + i/2, the
// compact first axis being even): nb holds the packed neighbours along the three compact
// axes (+1 side | -1 side << 16) and the cell itself, ca and cb the coefficients of the
// faces +x, -x, +y, -y and +z, -z, and 1 / diagonal.  A pass then reads its rows as three
// 16-byte LDS accesses per cell and computes no coordinates.
struct GArrays {
    double *phi, *rhs, *res, *inv, *sum;
    uint4* nb;
    float4 *ca, *cb;
    uint2* pw;  // per fine cell of an axis: parent | neighbour << 16, weight (FP32 bits)
    int* first;
};

// Carves the arrays from the workgroup's LDS (sub_bytes() of it); o: bytes used.  Offsets from
// the LDS array itself, so that the compiler sees LDS addresses (through integer casts the
// accesses became flat ones, three times slower).
__device__ __forceinline__ GArrays carve(char* lds, int& o, const GSub& G, int scratch) {
    GArrays A;
    const int c = G.cells;
    A.nb = (uint4*)lds;
    A.ca = (float4*)(lds + 16 * c);
    A.cb = (float4*)(lds + 32 * c);
    A.phi = (double*)(lds + 48 * c);
    A.rhs = (double*)(lds + 56 * c);
    o = 64 * c;
    A.inv = (double*)(lds + o);
    o += kDirect * kDirect * 8;
    A.sum = (double*)(lds + o);
    o += 64 * 8;
    A.res = (double*)(lds + o);
    o += max((scratch + 1) & ~1, kDirect * kDirect) * 8;
    A.pw = (uint2*)(lds + o);
    o += G.npn * 8;
    A.first = (int*)(lds + o);
    o = (o + G.nfirst * 4 + 15) & ~15;
    return A;
}

__device__ __forceinline__ void load_tables(const GArrays& A, const GSub& G, const GTab& t, int tid, int nt) {
    for (int k = tid; k < G.npn; k += nt)
        A.pw[k] = make_uint2(t.pn[G.pn0 + k], __float_as_uint(t.w[G.pn0 + k]));
    for (int k = tid; k < G.nfirst; k += nt) A.first[k] = t.first[G.first0 + k];
}

// The threads that work on a grid: the whole workgroup, or one wavefront of it (WAVE), which
// needs no barrier: its LDS accesses execute in order.
template <bool WAVE>
__device__ __forceinline__ void gsync() {
    if (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

__device__ __forceinline__ double row_off(const double* p, const uint4& q, const float4& a, const float4& b) {
    return (double)a.x * p[q.x & 0xffffu] + (double)a.y * p[q.x >> 16] + (double)a.z * p[q.y & 0xffffu] +
           (double)a.w * p[q.y >> 16] + (double)b.x * p[q.z & 0xffffu] + (double)b.y * p[q.z >> 16];
}

template <bool WAVE>
__device__ __forceinline__ void lds_sweeps(const GLds& L, const GArrays& A, int sweeps, double omega, int tid, int nt) {
    const int half = L.n >> 1;
    double* phi = A.phi + L.off;
    const double* rhs = A.rhs + L.off;
    for (int s = 0; s < 2 * sweeps; ++s) {
        const int o = L.off + (s & 1) * half;
        for (int h = tid; h < half; h += nt) {
            const uint4 q = A.nb[o + h];
            const float4 a = A.ca[o + h], b = A.cb[o + h];
            const double off = row_off(phi, q, a, b), p = phi[q.w];
            phi[q.w] = p + omega * ((off + rhs[q.w]) * (double)b.z - p);
        }
        gsync<WAVE>();
    }
}

// Sum of v(a, b, c) over a < na, b < nb, c < nc, each count 1 to 3: the eight terms of a run
// of two along each axis are fetched together, the rest of a longer run after them.
template <typename Fn>
__device__ __forceinline__ double sum_box(int na, int nb, int nc, Fn&& v) {
    double s = 0.0;
    double e[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int a = k & 1, b = (k >> 1) & 1, c = k >> 2;
        e[k] = (a < na && b < nb && c < nc) ? v(a, b, c) : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) s += e[k];
    if (na > 2 || nb > 2 || nc > 2)
        for (int c = 0; c < nc; ++c)
            for (int b = 0; b < nb; ++b)
                for (int a = (b < 2 && c < 2) ? 2 : 0; a < na; ++a) s += v(a, b, c);
    return s;
}

// Sum over the children of coarse cell (I, J, K) of grid C of the fine array r.
__device__ __forceinline__ double child_sum(const GLds& C, const GArrays& A, const double* r, int fx, int fxy, int I,
                                            int J, int K) {
    const int x0 = A.first[C.oc[0] + I], x1 = A.first[C.oc[0] + I + 1];
    const int y0 = A.first[C.oc[1] + J], y1 = A.first[C.oc[1] + J + 1];
    const int z0 = A.first[C.oc[2] + K], z1 = A.first[C.oc[2] + K + 1];
    const double* p = r + x0 + fx * y0 + fxy * z0;
    return sum_box(x1 - x0, y1 - y0, z1 - z0, [&](int a, int b, int c) { return p[a + fx * b + fxy * c]; });
}

template <bool WAVE>
__device__ __forceinline__ void lds_restrict(const GLds& C, const GArrays& A, int fx, int fy, int tid, int nt) {
    for (int t = tid; t < C.n; t += nt) {
        const int row = fdiv(t, C.inv_nx), I = t - row * C.nx, K = fdiv(row, C.inv_ny), J = row - K * C.ny;
        A.rhs[C.off + t] = child_sum(C, A, A.res, fx, fx * fy, I, J, K);
        A.phi[C.off + t] = 0.0;
    }
    gsync<WAVE>();
}

// Linear interpolation of grid C's correction at the fine cell (x, y, z).
__device__ __forceinline__ double interp(const GLds& C, const GArrays& A, int x, int y, int z) {
    const uint2 px = A.pw[C.of[0] + x], py = A.pw[C.of[1] + y], pz = A.pw[C.of[2] + z];
    const double wx = __uint_as_float(px.y), wy = __uint_as_float(py.y), wz = __uint_as_float(pz.y);
    const int x0 = px.x & 0xffffu, x1 = px.x >> 16, cxy = C.nx * C.ny;
    const int y0 = C.nx * (int)(py.x & 0xffffu), y1 = C.nx * (int)(py.x >> 16);
    const int z0 = cxy * (int)(pz.x & 0xffffu), z1 = cxy * (int)(pz.x >> 16);
    const double* p = A.phi + C.off;
    auto line = [&](int o) { return p[o + x0] + wx * (p[o + x1] - p[o + x0]); };
    const double a = line(y0 + z0), b = line(y1 + z0), c = line(y0 + z1), d = line(y1 + z1);
    const double lo = a + wy * (b - a), hi = c + wy * (d - c);
    return lo + wz * (hi - lo);
}

template <bool WAVE>
__device__ __forceinline__ void lds_down(const GSub& G, int l, const GArrays& A, const GShape& sh, int tid, int nt) {
    const GLds& L = G.L[l];
    lds_sweeps<WAVE>(L, A, sh.pre, sh.omega, tid, nt);
    const double* phi = A.phi + L.off;
    for (int e = tid; e < L.n; e += nt) {
        const uint4 q = A.nb[L.off + e];
        const float4 a = A.ca[L.off + e], b = A.cb[L.off + e];
        const double diag = (double)a.x + (double)a.y + (double)a.z + (double)a.w + (double)b.x + (double)b.y;
        A.res[q.w] = A.rhs[L.off + q.w] + row_off(phi, q, a, b) - diag * phi[q.w];
    }
    gsync<WAVE>();
    lds_restrict<WAVE>(G.L[l + 1], A, L.nx, L.ny, tid, nt);
}

template <bool WAVE>
__device__ __forceinline__ void lds_up(const GSub& G, int l, const GArrays& A, const GShape& sh, int tid, int nt) {
    const GLds& L = G.L[l];
    for (int i = tid; i < L.n; i += nt) {
        const int row = fdiv(i, L.inv_nx), x = i - row * L.nx, z = fdiv(row, L.inv_ny), y = row - z * L.ny;
        A.phi[L.off + i] += interp(G.L[l + 1], A, x, y, z);
    }
    gsync<WAVE>();
    lds_sweeps<WAVE>(L, A, sh.post, sh.omega, tid, nt);
}

// The coarsest grid's correction from its inverse, by one wavefront: two lanes per cell.
__device__ __forceinline__ void lds_direct(const GLds& L, const GArrays& A, int lane) {
    const int i = lane & (kDirect - 1), h = lane / kDirect, n = L.n;
    double s = 0.0;
    for (int j = h; j < n; j += 64 / kDirect) s += A.inv[j * kDirect + i] * A.rhs[L.off + j];
#pragma unroll
    for (int m = kDirect; m < 64; m <<= 1) s += __shfl_xor(s, m, 64);
    if (lane < n) A.phi[L.off + lane] = s;
    gsync<true>();
}

// One V-cycle on the grids of G from a zero correction; grids of at most kWaveCells cells
// are left to the first wavefront, whose steps need no workgroup barrier.
constexpr int kWaveCells = 128;

__device__ __forceinline__ void lds_vcycle(const GSub& G, const GArrays& A, const GShape& sh, int tid, int nt) {
    const int last = G.nl - 1;
    int lw = 0;
    while (lw < last && G.L[lw].n > kWaveCells) ++lw;  // the last grid has at most kDirect cells
    for (int l = 0; l < lw; ++l) lds_down<false>(G, l, A, sh, tid, nt);
    if (tid < 64) {
        for (int l = lw; l < last; ++l) lds_down<true>(G, l, A, sh, tid, 64);
        lds_direct(G.L[last], A, tid);
        for (int l = last - 1; l >= lw; --l) lds_up<true>(G, l, A, sh, tid, 64);
    }
    __syncthreads();
    for (int l = lw - 1; l >= 0; --l) lds_up<false>(G, l, A, sh, tid, nt);
}

// Colour-ordered place of cell t = (x, y, z) of grid L.
__device__ __forceinline__ int lds_place(const GLds& L, int t, int x, int y, int z) {
    return ((x + y + z) & 1 ? L.n >> 1 : 0) + (t >> 1);
}

// Face coefficients of grid C towards the next cell of each axis, from a fine grid whose
// face of cell (x, y, z) along axis k is face(k, x, y, z).
template <typename FaceFn>
__device__ __forceinline__ void lds_coarsen(const GLds& C, const GArrays& A, const float* ratio, FaceFn&& face, int tid,
                                            int nt) {
    for (int t = tid; t < C.n; t += nt) {
        const int row = fdiv(t, C.inv_nx), I = t - row * C.nx, K = fdiv(row, C.inv_ny), J = row - K * C.ny;
        const int x0 = A.first[C.oc[0] + I], x1 = A.first[C.oc[0] + I + 1];
        const int y0 = A.first[C.oc[1] + J], y1 = A.first[C.oc[1] + J + 1];
        const int z0 = A.first[C.oc[2] + K], z1 = A.first[C.oc[2] + K + 1];
        double sx = 0.0, sy = 0.0, sz = 0.0;
        if (C.nx > 1)
            sx = sum_box(1, y1 - y0, z1 - z0, [&](int, int b, int c) { return face(0, x1 - 1, y0 + b, z0 + c); });
        if (C.ny > 1)
            sy = sum_box(x1 - x0, 1, z1 - z0, [&](int a, int, int c) { return face(1, x0 + a, y1 - 1, z0 + c); });
        if (C.nz > 1)
            sz = sum_box(x1 - x0, y1 - y0, 1, [&](int a, int b, int) { return face(2, x0 + a, y0 + b, z1 - 1); });
        const float cx = (float)(sx * (double)ratio[C.oc[0] + I]), cy = (float)(sy * (double)ratio[C.oc[1] + J]),
                    cz = (float)(sz * (double)ratio[C.oc[2] + K]);
        const int e = C.off + lds_place(C, t, I, J, K);
        A.ca[e].x = C.lead == 0 ? cx : (C.lead == 1 ? cy : cz);
        A.ca[e].z = C.lead == 0 ? cy : (C.lead == 1 ? cz : 0.0f);
        A.cb[e].x = C.lead == 0 ? cz : 0.0f;
    }
    __syncthreads();
}

// The rest of grid C's rows: neighbours, the faces towards the previous cells, 1 / diagonal.
__device__ __forceinline__ void lds_rows(const GLds& L, const GArrays& A, int tid, int nt) {
    const int ex = L.ex, ey = L.ey, ez = L.ez, exy = ex * ey;
    const float inv_ex = 1.0f / ex;
    for (int i = tid; i < L.n; i += nt) {
        const int row = fdiv(i, inv_ex), x = i - row * ex, z = fdiv(row, L.inv_ey), y = row - z * ey;
        const int xm = x == 0 ? i + ex - 1 : i - 1, xp = x == ex - 1 ? i - (ex - 1) : i + 1;
        const int ym = y == 0 ? i + exy - ex : i - ex, yp = y == ey - 1 ? i - (exy - ex) : i + ex;
        const int zm = z == 0 ? i + exy * (ez - 1) : i - exy, zp = z == ez - 1 ? i - exy * (ez - 1) : i + exy;
        const int e = L.off + lds_place(L, i, x, y, z);
        A.nb[e] = make_uint4((uint32_t)xp | ((uint32_t)xm << 16), (uint32_t)yp | ((uint32_t)ym << 16),
                             (uint32_t)zp | ((uint32_t)zm << 16), (uint32_t)i);
        const float ax = A.ca[L.off + lds_place(L, xm, x == 0 ? ex - 1 : x - 1, y, z)].x;
        const float ay = A.ca[L.off + lds_place(L, ym, x, y == 0 ? ey - 1 : y - 1, z)].z;
        const float az = A.cb[L.off + lds_place(L, zm, x, y, z == 0 ? ez - 1 : z - 1)].x;
        A.ca[e].y = ax;
        A.ca[e].w = ay;
        A.cb[e].y = az;
        const double d = (double)A.ca[e].x + (double)ax + (double)A.ca[e].z + (double)ay + (double)A.cb[e].x + (double)az;
        A.cb[e].z = d > 0.0 ? (float)(1.0 / d) : 0.0f;
    }
    __syncthreads();
}

// The coarser grids of G from grid 0's faces, every grid's rows, and the coarsest grid's
// inverse: Gauss-Jordan on its matrix plus a constant, which makes the singular operator
// (constants in its kernel) invertible and leaves its action on zero-sum right-hand sides.
// It is built in the scratch residuals and A.inv in turn, one barrier per step.
template <int NT>
__device__ __forceinline__ void lds_build(const GSub& G, const GArrays& A, const float* ratio, double* other, int tid) {
    constexpr int nt = NT;
    for (int l = 0; l < G.nl; ++l) {
        const GLds& L = G.L[l];
        lds_rows(L, A, tid, nt);
        if (l + 1 == G.nl) break;
        lds_coarsen(
            G.L[l + 1], A, ratio,
            [&](int k, int x, int y, int z) -> double {
                const int i = x + L.nx * (y + L.ny * z), e = L.off + lds_place(L, i, x, y, z), s = k - L.lead;
                return s == 0 ? A.ca[e].x : (s == 1 ? A.ca[e].z : (s == 2 ? A.cb[e].x : 0.0f));
            },
            tid, nt);
    }
    const GLds& L = G.L[G.nl - 1];
    const int n = L.n;
    constexpr int kR = kDirect * kDirect / NT;  // entries per thread
    double *from = (n & 1) ? other : A.inv, *to = (n & 1) ? A.inv : other;  // n steps end in A.inv
    double trace = 0.0;
    for (int e = 0; e < n; ++e) trace += 1.0 / (double)fmaxf(A.cb[L.off + e].z, 1e-30f);
    const double shift = trace / ((double)n * n);
    for (int e = tid; e < kDirect * kDirect; e += nt) from[e] = shift;
    __syncthreads();
    if (tid < n) {  // a row each
        const uint4 q = A.nb[L.off + tid];
        const float4 a = A.ca[L.off + tid], b = A.cb[L.off + tid];
        double* r = from + (int)q.w * kDirect;
        r[q.w] += (double)a.x + (double)a.y + (double)a.z + (double)a.w + (double)b.x + (double)b.y;
        r[q.x & 0xffffu] -= (double)a.x;
        r[q.x >> 16] -= (double)a.y;
        r[q.y & 0xffffu] -= (double)a.z;
        r[q.y >> 16] -= (double)a.w;
        r[q.z & 0xffffu] -= (double)b.x;
        r[q.z >> 16] -= (double)b.y;
    }
    for (int k = 0; k < n; ++k) {
        __syncthreads();
        const double piv = from[k * kDirect + k];
        double p = __builtin_amdgcn_rcp(piv);  // the inverse is part of the preconditioner: two
        p = p * (2.0 - piv * p);               // Newton steps bring the reciprocal to FP64
        p = p * (2.0 - piv * p);
        const double u = from[k * kDirect + (tid & (kDirect - 1))];
        double c[kR], v[kR];
#pragma unroll
        for (int r = 0; r < kR; ++r) {
            const int e = tid + r * NT;
            c[r] = from[(e & ~(kDirect - 1)) + k];
            v[r] = from[e];
        }
        const bool ik = (tid & (kDirect - 1)) == k;
#pragma unroll
        for (int r = 0; r < kR; ++r) {
            const int e = tid + r * NT;
            const double w = e / kDirect == k ? (ik ? p : u * p) : (ik ? -c[r] * p : v[r] - c[r] * (u * p));
            to[e] = w;
        }
        double* t = from;
        from = to;
        to = t;
    }
    __syncthreads();
}

// Sum of v over the workgroup, in every thread; fixed order.
__device__ __forceinline__ double wg_sum(double v, double* sm, int tid, int nt) {
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v += __shfl_down(v, s, 64);
    if ((tid & 63) == 0) sm[tid >> 6] = v;
    __syncthreads();
    double a = 0.0;
    for (int w = 0; w < nt / 64; ++w) a += sm[w];
    __syncthreads();
    return a;
}

// ------------------------------------------------------------------------------------
// The whole solve of a small lattice in one workgroup.  Each thread owns NS sites for the
// whole call and keeps their rows (neighbours, face permittivities, source) in registers;
// LDS holds the potential, which neighbours read, and the coarse grids.  Bound by the
// latency of its passes (LDS reads, the FP64 chain, a barrier: about 0.4 us), where a
// launched pass costs 3 us.  A step of the 4 x 4 x 128 column in FP32 takes 108 us, 91 of
// them here (28 for the rows, the coarse grids and the inverse, 4.9 cycles of 12.7),
// against 2850 us with launched cycles; of 16^3 in FP64 161 against 269 us.
// ------------------------------------------------------------------------------------
// CLK: with its clock (a kernel of its own: the ticks cost the other one registers).
template <typename T, int NS, int NT, bool CLK>
__global__ __launch_bounds__(NT) void k_small_solve(Scalars S, Fields<T> F, GSub G, GTab tab, SmallArgs P) {
    extern __shared__ __align__(16) char lds_raw[];
    const int tid = threadIdx.x;
    constexpr int nt = NT;
    const int nd = (int)S.ndomain, nx = S.nx, ny = S.ny, nzd = S.z1 - S.z0 + 1, nxy = S.nxy;
    int used;
    const GArrays A = carve(lds_raw, used, G, nd);
    double* phi = (double*)(lds_raw + used);
    T* eps = (T*)A.res;  // until the rows are built
    const unsigned base = (unsigned)S.z0 * (unsigned)nxy;
    const float inv_nx = 1.0f / nx, inv_ny = 1.0f / ny, inv_hx = 1.0f / (nx >> 1);
    load_tables(A, G, tab, tid, nt);

    // the start of the solve: the potential held, or its extrapolation in time (the order as
    // ek_step chooses it: fixed, or the order whose last start residual was smaller)
    int order = 1;
    bool probe = false;
    if (P.step) {
        order = P.history;
        if (order == 0 && P.fixed > 0) order = 2;
        if (order == 0) {
            order = (int)P.ctl[kCtlOrder];
            const int other = 5 - order;
            if (P.ctl[kCtlRel0 + order - 2] > 0.0 && (P.ctl[kCtlRel0 + other - 2] == 0.0 || P.ctl[kCtlSince] >= 64.0)) {
                order = other;
                probe = true;
            }
        }
    }
    // place of site t in phi: colour-split where there are two colours, so that a pass reads
    // and writes consecutive values
    auto place = [&](int t, int x, int y, int z) {
        return S.ncolor == 2 ? ((x + y + z) & 1 ? nd >> 1 : 0) + (t >> 1) : t;
    };
    auto split = [&](int t) {
        const int rw = fdiv(t, inv_nx), z = fdiv(rw, inv_ny);
        return place(t, t - rw * nx, rw - z * ny, z);
    };
    double qs = 0.0;
    for (int t = tid; t < nd; t += nt) {
        const unsigned i = base + (unsigned)t;
        double v = F.phi[i];
        if (P.step) {
            const double p1 = v, p2 = P.prev[i];
            if (order == 2) v = 2.0 * p1 - p2;
            if (order >= 3) v = 3.0 * (p1 - p2) + P.prev2[i];
            P.prev2[i] = p2;
            P.prev[i] = p1;
        }
        phi[split(t)] = v;
        eps[t] = F.eps[i];
        qs += (double)F.q[i];
    }
    const double charge = wg_sum(qs, A.sum, tid, nt);
    const double mean = (charge + (S.walls ? (S.sigma0 + S.sigma1) * (double)nxy : 0.0)) / (double)nd;

    // The owned sites.  Two colours: slots 2k and 2k + 1 hold site tid + k nt of the red and
    // of the black ones; three colours: slot k holds site tid + k nt of the lattice.
    int own[NS], at[NS], col[NS];
    uint32_t nbx[NS], nby[NS], nbz[NS];
    double fxp[NS], fxm[NS], fyp[NS], fym[NS], fzp[NS], fzm[NS], idg[NS], src[NS];
    double ss = 0.0;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        int t, x, y, z;
        if (S.ncolor == 2) {
            const int h = tid + (k >> 1) * nt, c = k & 1;
            const int rw = fdiv(h, inv_hx), m = h - rw * (nx >> 1);
            z = fdiv(rw, inv_ny);
            y = rw - z * ny;
            x = 2 * m + ((c + y + z) & 1);
            t = h < nd / 2 ? x + nx * rw : -1;
            col[k] = c;
        } else {
            t = tid + k * nt;
            const int rw = fdiv(t, inv_nx);
            x = t - rw * nx;
            z = fdiv(rw, inv_ny);
            y = rw - z * ny;
            if (t >= nd) t = -1;
            const int cy = ((ny & 1) && ny >= 3 && y == ny - 1) ? 2 : (y & 1);
            const int cz = ((nzd & 1) && nzd >= 3 && !S.walls && z == nzd - 1) ? 2 : (z & 1);
            col[k] = ((x & 1) + cy + cz) % 3;
        }
        own[k] = t;
        at[k] = 0;
        nbx[k] = nby[k] = nbz[k] = 0;
        fxp[k] = fxm[k] = fyp[k] = fym[k] = fzp[k] = fzm[k] = idg[k] = src[k] = 0.0;
        if (t < 0) {
            col[k] = -1;
            continue;
        }
        const int xa = x == 0 ? t + nx - 1 : t - 1, xb = x == nx - 1 ? t - (nx - 1) : t + 1;
        const int ya = y == 0 ? t + nxy - nx : t - nx, yb = y == ny - 1 ? t - (nxy - nx) : t + nx;
        const int za = z == 0 ? t + nxy * (nzd - 1) : t - nxy, zb = z == nzd - 1 ? t - nxy * (nzd - 1) : t + nxy;
        at[k] = place(t, x, y, z);
        // two colours: every neighbour has the other one
        auto other = [&](int j) -> uint32_t {
            return S.ncolor == 2 ? (uint32_t)(((x + y + z) & 1 ? 0 : nd >> 1) + (j >> 1)) : (uint32_t)j;
        };
        nbx[k] = other(xb) | (other(xa) << 16);
        nby[k] = other(yb) | (other(ya) << 16);
        nbz[k] = other(zb) | (other(za) << 16);
        // a face that is left out (an axis of length 1, a wall) has a zero coefficient
        const double ei = eps[t];
        const bool ony = ny > 1, lo = nzd > 1 && !(S.walls && z == 0), hi = nzd > 1 && !(S.walls && z == nzd - 1);
        fxm[k] = 0.5 * (ei + (double)eps[xa]);
        fxp[k] = 0.5 * (ei + (double)eps[xb]);
        if (ony) fym[k] = 0.5 * (ei + (double)eps[ya]);
        if (ony) fyp[k] = 0.5 * (ei + (double)eps[yb]);
        if (lo) fzm[k] = 0.5 * (ei + (double)eps[za]);
        if (hi) fzp[k] = 0.5 * (ei + (double)eps[zb]);
        const double diag = (fxm[k] + fxp[k]) + (fym[k] + fyp[k]) + fzm[k] + fzp[k];
        idg[k] = diag > 0.0 ? 1.0 / diag : 0.0;
        double s = (double)F.q[base + (unsigned)t];
        if (S.walls && z == 0) s += S.sigma0;
        if (S.walls && z == nzd - 1) s += S.sigma1;
        if (S.polar) s -= S.E_ext[0] * (fxp[k] - fxm[k]) + S.E_ext[1] * (fyp[k] - fym[k]) + S.E_ext[2] * (fzp[k] - fzm[k]);
        src[k] = s - mean;
        ss += src[k] * src[k];
    }
    ss = wg_sum(ss, A.sum, tid, nt);
    if (G.nl > 0) {
        lds_coarsen(
            G.L[0], A, tab.ratio + G.first0,
            [&](int k, int x, int y, int z) -> double {
                const int t = x + nx * (y + ny * z);
                int j;
                if (k == 0)
                    j = x == nx - 1 ? t - (nx - 1) : t + 1;
                else if (k == 1)
                    j = y == ny - 1 ? t - (nxy - nx) : t + nx;
                else
                    j = z == nzd - 1 ? t - nxy * (nzd - 1) : t + nxy;
                return 0.5 * ((double)eps[t] + (double)eps[j]);
            },
            tid, nt);
        __syncthreads();  // the last reads of eps, whose place the build reuses
        lds_build<NT>(G, A, tab.ratio + G.first0, A.res, tid);
    }

    auto off_of = [&](int k) __attribute__((always_inline)) {
        return fxp[k] * phi[nbx[k] & 0xffffu] + fxm[k] * phi[nbx[k] >> 16] + fyp[k] * phi[nby[k] & 0xffffu] +
               fym[k] * phi[nby[k] >> 16] + fzp[k] * phi[nbz[k] & 0xffffu] + fzm[k] * phi[nbz[k] >> 16];
    };
    // residuals into A.res and the sum of their squares
    auto residual = [&]() __attribute__((always_inline)) {
        double rr = 0.0;
#pragma unroll
        for (int k = 0; k < NS; ++k)
            if (own[k] >= 0) {
                const double diag = (fxm[k] + fxp[k]) + (fym[k] + fyp[k]) + fzm[k] + fzp[k];
                const double r = src[k] + off_of(k) - diag * phi[at[k]];
                A.res[own[k]] = r;
                rr += r * r;
            }
        return wg_sum(rr, A.sum, tid, nt);
    };
    long long smoothing = 0;  // ticks in the lattice sweeps
    auto sweeps = [&](int n) __attribute__((always_inline)) {
        const long long t0 = CLK ? wall_clock64() : 0;
        for (int s = 0; s < n; ++s)
            for (int c = 0; c < S.ncolor; ++c) {
#pragma unroll
                for (int k = 0; k < NS; ++k)
                    if (col[k] == c) {
                        const double old = phi[at[k]], gs = (off_of(k) + src[k]) * idg[k];
                        if (idg[k] > 0.0) phi[at[k]] = old + P.sh.omega * (gs - old);
                    }
                __syncthreads();
            }
        if (CLK) smoothing += wall_clock64() - t0;
    };

    const double rr0 = residual();  // (its barriers: every thread is past the reads of eps)
    double rr = rr0;
    const double stop = P.tol * P.tol * ss, deep = P.margin * P.margin * stop;
    const int most = P.fixed > 0 ? P.fixed : P.maxit;
    // A cycle costs little here, and one taken beyond the tolerance leaves an error well below
    // it: over 5000 steps of the column the errors of solves that stop just short of the
    // tolerance add up to 2e-9 of the density.  A second one follows where the first does not reach
    // the margin of the launched cycles (2x2x300 in FP64: 7.5e-12 of phi after one, SOR 3.1e-12).
    int it = 0, beyond = 0;
    const long long started = CLK ? wall_clock64() : 0;
    while (ss > 0.0 && it < most && rr < 1e300) {  // (not finite: no cycle can mend it)
        if (P.fixed == 0 && rr <= stop) {
            if (it == 0 || beyond == 2 || (beyond == 1 && rr <= deep)) break;
            ++beyond;
        }
        sweeps(P.sh.fine_pre);
        if (G.nl > 0) {
            if (P.sh.fine_pre > 0) (void)residual();
            lds_restrict<false>(G.L[0], A, nx, ny, tid, nt);
            lds_vcycle(G, A, P.sh, tid, nt);
#pragma unroll
            for (int k = 0; k < NS; ++k)
                if (own[k] >= 0) {
                    const int t = own[k], rw = fdiv(t, inv_nx), z = fdiv(rw, inv_ny);
                    phi[at[k]] += interp(G.L[0], A, t - rw * nx, rw - z * ny, z);
                }
            __syncthreads();
        }
        sweeps(P.sh.fine_post);
        rr = residual();
        ++it;
    }
    if (CLK && tid == 0) {
        P.clock[kClkIter] += (double)(wall_clock64() - started);
        P.clock[kClkCycles] += it;
        P.clock[kClkSmooth] += (double)smoothing;
        P.clock[kClkPasses] += (double)it * (P.sh.fine_pre + P.sh.fine_post) * S.ncolor;
    }

    // gauge mean(phi) = 0 and the wall layers (Gauss's law at the charged wall faces)
    double ps = 0.0;
    for (int t = tid; t < nd; t += nt) ps += phi[t];
    const double shift = wg_sum(ps, A.sum, tid, nt) / (double)nd;
    const bool zero = !(ss > 0.0);
    for (int t = tid; t < nd; t += nt) {
        const double v = zero ? 0.0 : phi[split(t)] - shift;
        const unsigned i = base + (unsigned)t;
        F.phi[i] = v;
        if (S.walls && t < nxy) F.phi[i - nxy] = v + S.sigma0 / (double)F.eps[i];
        if (S.walls && t >= nd - nxy) F.phi[i + nxy] = v + S.sigma1 / (double)F.eps[i];
    }
    if (tid == 0) {
        const double rel = ss > 0.0 ? sqrt(rr / ss) : 0.0, rel0 = ss > 0.0 ? sqrt(rr0 / ss) : 0.0;
        F.scal[0] = mean;
        F.scal[1] = rr;
        F.scal[2] = ss;
        F.scal[24] = rr0;
        F.scal[25] = ss;
        if (P.step && P.fixed > 0) {  // the record ek_observables reads when nothing is read back
            F.scal[28] = fmax(F.scal[28], rel);
            F.scal[29] = rel;
            F.scal[30] = rel0;
        }
        double* c = P.ctl;
        c[kCtlIters] = it;
        c[kCtlTotal] += it;
        c[kCtlRel] = rel;
        c[kCtlRelStart] = rel0;
        c[kCtlRelMax] = fmax(c[kCtlRelMax], rel);
        if (P.fixed == 0 && rr > stop) c[kCtlNoConv] = 1.0;
        if (P.step) {
            if (P.history == 0 && P.fixed == 0 && c[kCtlSteps] >= 2.0) {
                c[kCtlRel0 + order - 2] = rel0;
                if (probe) {
                    c[kCtlSince] = 0.0;
                    if (rel0 < c[kCtlRel0 + 3 - order]) c[kCtlOrder] = order;
                } else {
                    c[kCtlSince] += 1.0;
                }
            }
            c[kCtlSteps] += 1.0;
        }
    }
}

template <typename T>
void launch_small_solve(const Scalars& S, const Fields<T>& F, const GSub& G, const GTab& t, const SmallArgs& a,
                        hipStream_t st) {
    const size_t lds = sub_bytes(G, S.ndomain) + (size_t)S.ndomain * 8;
    // Sites per thread and threads: 512 threads hold up to four rows each in registers; above
    // 2048 sites twice the threads (128 registers, a few spills) beat twice the rows (16^3 in
    // FP64: 152 against 156 us per step, 14 x 17 x 15 in FP32: 185 against 206).
    auto go = [&](auto kernel, int nt) { hipLaunchKernelGGL(kernel, dim3(1), dim3(nt), lds, st, S, F, G, t, a); };
    const bool clk = a.clock != nullptr;
    if (S.ndomain <= 1024)
        clk ? go(k_small_solve<T, 2, 512, true>, 512) : go(k_small_solve<T, 2, 512, false>, 512);
    else if (S.ndomain <= 2048)
        clk ? go(k_small_solve<T, 4, 512, true>, 512) : go(k_small_solve<T, 4, 512, false>, 512);
    else
        clk ? go(k_small_solve<T, 4, 1024, true>, 1024) : go(k_small_solve<T, 4, 1024, false>, 1024);
}

// ------------------------------------------------------------------------------------
// Launched grids: lattices above the single-workgroup size whose axes the V-cycle of
// ek_kernels.hip cannot halve to the end.  The lattice is smoothed by its colour passes in
// site order (three colours with an odd periodic axis) and the upper coarse grids by
// k_mg_smooth on their compact axes; the grids that fit one workgroup run in k_g_tail.
// These lattices took SOR before: 4 x 128 x 128 in FP64 319 sweeps a step, 2.9 ms.
// ------------------------------------------------------------------------------------
namespace {

__device__ __forceinline__ double* coef_of(const MGLevel& M, int lead, int k) {
    const int s = k - lead;
    return s == 0 ? M.ax : (s == 1 ? M.ay : M.az);
}

struct Box {
    int lo[3], hi[3];
};

// Coordinates of cell t of a grid, and its children.
__device__ __forceinline__ void cell_of(const GTrans& C, unsigned t, int& I, int& J, int& K) {
    const unsigned r = div_exact(t, C.inv_nx);
    I = (int)(t - r * (unsigned)C.d[0]);
    K = (int)div_exact(r, C.inv_ny);
    J = (int)(r - (unsigned)K * (unsigned)C.d[1]);
}

__device__ __forceinline__ Box children(const GTrans& C, const GTab& t, int I, int J, int K) {
    Box b;
    b.lo[0] = t.first[C.oc[0] + I], b.hi[0] = t.first[C.oc[0] + I + 1];
    b.lo[1] = t.first[C.oc[1] + J], b.hi[1] = t.first[C.oc[1] + J + 1];
    b.lo[2] = t.first[C.oc[2] + K], b.hi[2] = t.first[C.oc[2] + K + 1];
    return b;
}

// Stores the face coefficients of coarse cell t from the fine faces face(k, x, y, z).
template <typename FaceFn>
__device__ __forceinline__ void coarsen_cell(const GTrans& C, const MGLevel& M, const GTab& tab, unsigned t,
                                             FaceFn&& face) {
    int I, J, K;
    cell_of(C, t, I, J, K);
    const Box b = children(C, tab, I, J, K);
    double s[3] = {0.0, 0.0, 0.0};
    const int n0 = b.hi[0] - b.lo[0], n1 = b.hi[1] - b.lo[1], n2 = b.hi[2] - b.lo[2];
    if (C.d[0] > 1) s[0] = sum_box(1, n1, n2, [&](int, int y, int z) { return face(0, b.hi[0] - 1, b.lo[1] + y, b.lo[2] + z); });
    if (C.d[1] > 1) s[1] = sum_box(n0, 1, n2, [&](int x, int, int z) { return face(1, b.lo[0] + x, b.hi[1] - 1, b.lo[2] + z); });
    if (C.d[2] > 1) s[2] = sum_box(n0, n1, 1, [&](int x, int y, int) { return face(2, b.lo[0] + x, b.lo[1] + y, b.hi[2] - 1); });
    const double c0 = s[0] * (double)tab.ratio[C.oc[0] + I], c1 = s[1] * (double)tab.ratio[C.oc[1] + J],
                 c2 = s[2] * (double)tab.ratio[C.oc[2] + K];
    M.ax[t] = C.lead == 0 ? c0 : (C.lead == 1 ? c1 : c2);
    M.ay[t] = C.lead == 0 ? c1 : (C.lead == 1 ? c2 : 0.0);
    M.az[t] = C.lead == 0 ? c2 : 0.0;
}

// Row of cell i of a grid in its compact axes.
__device__ __forceinline__ void grid_row(const MGLevel& M, unsigned i, double& diag, double& off) {
    int x, y, z;
    level_xyz(i, M, x, y, z);
    const unsigned ex = (unsigned)M.nx, exy = ex * (unsigned)M.ny;
    const unsigned xm = x == 0 ? i + ex - 1 : i - 1, xp = x == M.nx - 1 ? i - (ex - 1) : i + 1;
    const unsigned ym = y == 0 ? i + exy - ex : i - ex, yp = y == M.ny - 1 ? i - (exy - ex) : i + ex;
    const unsigned zm = z == 0 ? i + exy * (unsigned)(M.nz - 1) : i - exy,
                   zp = z == M.nz - 1 ? i - exy * (unsigned)(M.nz - 1) : i + exy;
    const double a0 = M.ax[i], a1 = M.ax[xm], b0 = M.ay[i], b1 = M.ay[ym], c0 = M.az[i], c1 = M.az[zm];
    diag = a0 + a1 + b0 + b1 + c0 + c1;
    off = a0 * M.phi[xp] + a1 * M.phi[xm] + b0 * M.phi[yp] + b1 * M.phi[ym] + c0 * M.phi[zp] + c1 * M.phi[zm];
}

// Right-hand side of coarse cell t and the start of its correction: zero, or with
// red_omega > 0 on red cells the first red pass of the pre-smoothing, which from a zero
// correction is omega s / diag.
__device__ __forceinline__ void coarse_begin(const MGLevel& M, unsigned t, double s, double red_omega) {
    double v = 0.0;
    if (red_omega > 0.0) {
        int x, y, z;
        level_xyz(t, M, x, y, z);
        if (((x + y + z) & 1) == 0) {
            const unsigned ex = (unsigned)M.nx, exy = ex * (unsigned)M.ny;
            const unsigned xm = x == 0 ? t + ex - 1 : t - 1, ym = y == 0 ? t + exy - ex : t - ex,
                           zm = z == 0 ? t + exy * (unsigned)(M.nz - 1) : t - exy;
            const double d = M.ax[t] + M.ax[xm] + M.ay[t] + M.ay[ym] + M.az[t] + M.az[zm];
            if (d > 0.0) v = red_omega * (s / d);
        }
    }
    M.s[t] = s;
    M.phi[t] = v;
}

// Sum over the children of coarse cell t by eight lanes, lane (a, b, c) taking every other
// child along each axis; in lane 0.
template <typename Fn>
__device__ __forceinline__ double restrict_cell(const GTrans& C, const GTab& tab, unsigned t, int lane, Fn&& residual) {
    int I, J, K;
    cell_of(C, t, I, J, K);
    const Box b = children(C, tab, I, J, K);
    double s = 0.0;
    for (int z = b.lo[2] + (lane >> 2); z < b.hi[2]; z += 2)
        for (int y = b.lo[1] + ((lane >> 1) & 1); y < b.hi[1]; y += 2)
            for (int x = b.lo[0] + (lane & 1); x < b.hi[0]; x += 2) s += residual(x, y, z);
#pragma unroll
    for (int m = 4; m > 0; m >>= 1) s += __shfl_down(s, m, 8);
    return s;
}

__device__ __forceinline__ double interp_at(const GTrans& C, const MGLevel& M, const GTab& t, int x, int y, int z) {
    const uint32_t px = t.pn[C.of[0] + x], py = t.pn[C.of[1] + y], pz = t.pn[C.of[2] + z];
    const double wx = t.w[C.of[0] + x], wy = t.w[C.of[1] + y], wz = t.w[C.of[2] + z];
    const unsigned x0 = px & 0xffffu, x1 = px >> 16, cx = (unsigned)C.d[0], cxy = cx * (unsigned)C.d[1];
    const unsigned y0 = cx * (py & 0xffffu), y1 = cx * (py >> 16), z0 = cxy * (pz & 0xffffu), z1 = cxy * (pz >> 16);
    const double* p = M.phi;
    auto line = [&](unsigned o) { return p[o + x0] + wx * (p[o + x1] - p[o + x0]); };
    const double a = line(y0 + z0), b = line(y1 + z0), c = line(y0 + z1), d = line(y1 + z1);
    const double lo = a + wy * (b - a), hi = c + wy * (d - c);
    return lo + wz * (hi - lo);
}

// Domain site of lattice coordinates (z counted from the first domain layer).
__device__ __forceinline__ unsigned domain_site(const Scalars& S, int x, int y, int z) {
    return (unsigned)x + (unsigned)S.nx * ((unsigned)y + (unsigned)S.ny * (unsigned)(z + S.z0));
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_g_coarsen0(Scalars S, Fields<T> F, GTrans C, MGLevel M, GTab tab) {
    const unsigned t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= C.n) return;
    const int nzd = S.z1 - S.z0 + 1;
    coarsen_cell(C, M, tab, t, [&](int k, int x, int y, int z) {
        const int x2 = k == 0 ? (x + 1 == S.nx ? 0 : x + 1) : x, y2 = k == 1 ? (y + 1 == S.ny ? 0 : y + 1) : y,
                  z2 = k == 2 ? (z + 1 == nzd ? 0 : z + 1) : z;
        return 0.5 * ((double)F.eps[domain_site(S, x, y, z)] + (double)F.eps[domain_site(S, x2, y2, z2)]);
    });
}

__global__ __launch_bounds__(kBlock) void k_g_coarsen(GTrans Cf, MGLevel Mf, GTrans C, MGLevel M, GTab tab) {
    const unsigned t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= C.n) return;
    coarsen_cell(C, M, tab, t, [&](int k, int x, int y, int z) {
        return coef_of(Mf, Cf.lead, k)[(unsigned)x + (unsigned)Cf.d[0] * ((unsigned)y + (unsigned)Cf.d[1] * (unsigned)z)];
    });
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_g_restrict0(Scalars S, Fields<T> F, GTrans C, MGLevel M, GTab tab,
                                                        double red_omega) {
    const unsigned u = blockIdx.x * kBlock + threadIdx.x, t = u >> 3;
    if (t >= C.n) return;  // groups of eight lanes leave together
    const double mean = F.scal[0];
    const int nzd = S.z1 - S.z0 + 1;
    const double s = restrict_cell(C, tab, t, (int)(u & 7u), [&](int x, int y, int z) {
        const unsigned i = domain_site(S, x, y, z), nx = (unsigned)S.nx, nxy = (unsigned)S.nxy;
        const unsigned xa = x == 0 ? i + nx - 1 : i - 1, xb = x == S.nx - 1 ? i - (nx - 1) : i + 1;
        const unsigned ya = y == 0 ? i + nxy - nx : i - nx, yb = y == S.ny - 1 ? i - (nxy - nx) : i + nx;
        const unsigned za = z == 0 ? i + nxy * (unsigned)(nzd - 1) : i - nxy,
                       zb = z == nzd - 1 ? i - nxy * (unsigned)(nzd - 1) : i + nxy;
        const bool ony = S.ny > 1, lo = nzd > 1 && !(S.walls && z == 0), hi = nzd > 1 && !(S.walls && z == nzd - 1);
        const double ei = F.eps[i], p = F.phi[i];
        const double fxm = 0.5 * (ei + (double)F.eps[xa]), fxp = 0.5 * (ei + (double)F.eps[xb]);
        const double fym = ony ? 0.5 * (ei + (double)F.eps[ya]) : 0.0, fyp = ony ? 0.5 * (ei + (double)F.eps[yb]) : 0.0;
        const double fzm = lo ? 0.5 * (ei + (double)F.eps[za]) : 0.0, fzp = hi ? 0.5 * (ei + (double)F.eps[zb]) : 0.0;
        double src = (double)F.q[i];
        if (S.walls && z == 0) src += S.sigma0;
        if (S.walls && z == nzd - 1) src += S.sigma1;
        if (S.polar) src -= S.E_ext[0] * (fxp - fxm) + S.E_ext[1] * (fyp - fym) + S.E_ext[2] * (fzp - fzm);
        return (src - mean) + fxp * (F.phi[xb] - p) + fxm * (F.phi[xa] - p) + fyp * (F.phi[yb] - p) +
               fym * (F.phi[ya] - p) + fzp * (F.phi[zb] - p) + fzm * (F.phi[za] - p);
    });
    if ((u & 7u) == 0) coarse_begin(M, t, s, red_omega);
}

__global__ __launch_bounds__(kBlock) void k_g_restrict(GTrans Cf, MGLevel Mf, GTrans C, MGLevel M, GTab tab,
                                                       double red_omega) {
    const unsigned u = blockIdx.x * kBlock + threadIdx.x, t = u >> 3;
    if (t >= C.n) return;
    const double s = restrict_cell(C, tab, t, (int)(u & 7u), [&](int x, int y, int z) {
        const unsigned i = (unsigned)x + (unsigned)Cf.d[0] * ((unsigned)y + (unsigned)Cf.d[1] * (unsigned)z);
        double diag, off;
        grid_row(Mf, i, diag, off);
        return Mf.s[i] + off - diag * Mf.phi[i];
    });
    if ((u & 7u) == 0) coarse_begin(M, t, s, red_omega);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_g_prolong0(Scalars S, Fields<T> F, GTrans C, MGLevel M, GTab tab) {
    const unsigned t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= S.ndomain) return;
    const unsigned i = t + (unsigned)S.z0 * (unsigned)S.nxy;
    int x, y, z;
    site_xyz(i, S, x, y, z);
    F.phi[i] += interp_at(C, M, tab, x, y, z - S.z0);
}

__global__ __launch_bounds__(kBlock) void k_g_prolong(GTrans Cf, MGLevel Mf, GTrans C, MGLevel M, GTab tab) {
    const unsigned t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= Cf.n) return;
    int x, y, z;
    cell_of(Cf, t, x, y, z);
    Mf.phi[t] += interp_at(C, M, tab, x, y, z);
}

constexpr int kTailGThreads = 512;

// Rows of the grids that k_g_tail holds and the coarsest one's inverse, once per solve, from
// the first of them's coefficients (M); kept in `rows` as k_g_tail loads them.
__global__ __launch_bounds__(kTailGThreads) void k_g_tail_build(GSub G, GTab tab, MGLevel M, uint4* rows) {
    extern __shared__ __align__(16) char lds_raw[];
    const int tid = threadIdx.x;
    constexpr int nt = kTailGThreads;
    int used;
    const GArrays A = carve(lds_raw, used, G, G.L[0].n);
    load_tables(A, G, tab, tid, nt);
    const GLds& L = G.L[0];
    const float inv_ex = 1.0f / L.ex;
    for (int i = tid; i < L.n; i += nt) {
        const int row = fdiv(i, inv_ex), x = i - row * L.ex, z = fdiv(row, L.inv_ey), y = row - z * L.ey;
        const int e = lds_place(L, i, x, y, z);
        A.ca[e].x = (float)M.ax[i];
        A.ca[e].z = (float)M.ay[i];
        A.cb[e].x = (float)M.az[i];
    }
    __syncthreads();
    lds_build<nt>(G, A, tab.ratio + G.first0, A.res, tid);
    const uint4* all = A.nb;  // nb, ca, cb and inv lie one after another but for phi and rhs
    for (int k = tid; k < 3 * G.cells; k += nt) rows[k] = all[k];
    double* inv = (double*)(rows + 3 * G.cells);
    for (int k = tid; k < kDirect * kDirect; k += nt) inv[k] = A.inv[k];
}

// One V-cycle on the grids of G for the right-hand side M.s; the correction goes to M.phi.
__global__ __launch_bounds__(kTailGThreads) void k_g_tail(GSub G, GTab tab, MGLevel M, const uint4* rows, GShape sh) {
    extern __shared__ __align__(16) char lds_raw[];
    const int tid = threadIdx.x;
    constexpr int nt = kTailGThreads;
    int used;
    const GArrays A = carve(lds_raw, used, G, G.L[0].n);
    uint4* all = A.nb;
    for (int k = tid; k < 3 * G.cells; k += nt) all[k] = rows[k];
    const double* inv = (const double*)(rows + 3 * G.cells);
    for (int k = tid; k < kDirect * kDirect; k += nt) A.inv[k] = inv[k];
    load_tables(A, G, tab, tid, nt);
    for (int i = tid; i < G.L[0].n; i += nt) {
        A.rhs[i] = M.s[i];
        A.phi[i] = 0.0;
    }
    __syncthreads();
    lds_vcycle(G, A, sh, tid, nt);
    for (int i = tid; i < G.L[0].n; i += nt) M.phi[i] = A.phi[i];
}

unsigned blocks_of(unsigned n) { return (n + kBlock - 1) / kBlock; }

}  // namespace

size_t gmg_rows_bytes(const GSub& G) { return (size_t)G.cells * 48 + kDirect * kDirect * 8; }

template <typename T>
void launch_g_coarsen0(const Scalars& S, const Fields<T>& F, const GTrans& C, const MGLevel& M, const GTab& t,
                       hipStream_t st) {
    hipLaunchKernelGGL(k_g_coarsen0<T>, dim3(blocks_of(C.n)), dim3(kBlock), 0, st, S, F, C, M, t);
}
void launch_g_coarsen(const GTrans& Cf, const MGLevel& Mf, const GTrans& C, const MGLevel& M, const GTab& t,
                      hipStream_t st) {
    hipLaunchKernelGGL(k_g_coarsen, dim3(blocks_of(C.n)), dim3(kBlock), 0, st, Cf, Mf, C, M, t);
}
template <typename T>
void launch_g_restrict0(const Scalars& S, const Fields<T>& F, const GTrans& C, const MGLevel& M, const GTab& t,
                        double red_omega, hipStream_t st) {
    hipLaunchKernelGGL(k_g_restrict0<T>, dim3(blocks_of(8 * C.n)), dim3(kBlock), 0, st, S, F, C, M, t, red_omega);
}
void launch_g_restrict(const GTrans& Cf, const MGLevel& Mf, const GTrans& C, const MGLevel& M, const GTab& t,
                       double red_omega, hipStream_t st) {
    hipLaunchKernelGGL(k_g_restrict, dim3(blocks_of(8 * C.n)), dim3(kBlock), 0, st, Cf, Mf, C, M, t, red_omega);
}
template <typename T>
void launch_g_prolong0(const Scalars& S, const Fields<T>& F, const GTrans& C, const MGLevel& M, const GTab& t,
                       hipStream_t st) {
    hipLaunchKernelGGL(k_g_prolong0<T>, dim3(blocks_of(S.ndomain)), dim3(kBlock), 0, st, S, F, C, M, t);
}
void launch_g_prolong(const GTrans& Cf, const MGLevel& Mf, const GTrans& C, const MGLevel& M, const GTab& t,
                      hipStream_t st) {
    hipLaunchKernelGGL(k_g_prolong, dim3(blocks_of(Cf.n)), dim3(kBlock), 0, st, Cf, Mf, C, M, t);
}
void launch_g_tail_build(const GSub& G, const GTab& t, const MGLevel& M, void* rows, hipStream_t st) {
    hipLaunchKernelGGL(k_g_tail_build, dim3(1), dim3(kTailGThreads), tail_bytes(G), st, G, t, M, (uint4*)rows);
}
void launch_g_tail(const GSub& G, const GTab& t, const MGLevel& M, const void* rows, const GShape& sh, hipStream_t st) {
    hipLaunchKernelGGL(k_g_tail, dim3(1), dim3(kTailGThreads), tail_bytes(G), st, G, t, M, (const uint4*)rows, sh);
}

#define EK_GMG_INST(T)                                                                                                 \
    template void launch_small_solve<T>(const Scalars&, const Fields<T>&, const GSub&, const GTab&, const SmallArgs&,  \
                                        hipStream_t);                                                                  \
    template void launch_g_coarsen0<T>(const Scalars&, const Fields<T>&, const GTrans&, const MGLevel&, const GTab&,   \
                                       hipStream_t);                                                                   \
    template void launch_g_restrict0<T>(const Scalars&, const Fields<T>&, const GTrans&, const MGLevel&, const GTab&,  \
                                        double, hipStream_t);                                                          \
    template void launch_g_prolong0<T>(const Scalars&, const Fields<T>&, const GTrans&, const MGLevel&, const GTab&,   \
                                       hipStream_t);
EK_GMG_INST(float)
EK_GMG_INST(double)

}  // namespace ek
