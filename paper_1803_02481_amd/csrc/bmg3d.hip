// bmg3d.hip -- the 3D path of hipbmg: finite volumes, operator-induced
// interpolation, 27-point Galerkin coarse operators, eight-colour Gauss-Seidel
// V(nu1,nu2)-cycles and the coarsest Cholesky solve (section 2, Algorithm 1;
// section 3: interpolation in 3D, the r/C term, the coarse solve), and the C
// interface declared in include/hipbmg3d.h.
//
// Octant layout.  A level of nx x ny x nz vertices holds every field as eight
// sub-grids, octant o = (i&1) + 2(j&1) + 4(k&1), each mx x my x mz with
// mx = (nx+1)/2 (the odd octants leave their last entry unused), rows pitched
// to px = mx rounded up to 8.  Vertex (i,j,k) sits at
//   o * oct + (k>>1) * plane + (j>>1) * px + (i>>1).
// So one colour of the relaxation is one contiguous sub-grid, its neighbours
// in direction d are the sub-grid of octant o ^ (odd bits of d) shifted by 0
// or -1/+1 rows, and the next coarser level is octant 0 itself.  The kinds of
// fine vertex in the interpolation are octants as well: 0 coarse points,
// 1, 2, 4 on coarse lines, 3, 5, 6 on coarse faces, 7 cell centres; each
// keeps its weights in 2, 4 or 8 octant-sized slots (26 in all).
#include "hipbmg3d.h"
#include "bmg_internal.h"
#include "bmg_model.h"
#include "bmg_quot.h"
#include "bmg_tags.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

namespace {

using hbmg::div_by;

// ---------------------------------------------------------------------------
// geometry
// ---------------------------------------------------------------------------
struct Oct {
    int nx, ny, nz;
    int mx, my, mz, px;
    long long plane, oct, field;
};

Oct make_oct(int nx, int ny, int nz)
{
    Oct g;
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.mx = (nx + 1) / 2;
    g.my = (ny + 1) / 2;
    g.mz = (nz + 1) / 2;
    g.px = (g.mx + 7) & ~7;
    g.plane = (long long)g.px * g.my;
    g.oct = g.plane * g.mz;
    g.field = 8 * g.oct;
    return g;
}

__host__ __device__ inline int oct_of(int i, int j, int k) { return (i & 1) | ((j & 1) << 1) | ((k & 1) << 2); }

__host__ __device__ inline long long sub_of(const Oct &g, int i, int j, int k)
{
    return (long long)(k >> 1) * g.plane + (long long)(j >> 1) * g.px + (i >> 1);
}

__host__ __device__ inline long long vid(const Oct &g, int i, int j, int k)
{
    return oct_of(i, j, k) * g.oct + sub_of(g, i, j, k);
}

__host__ __device__ inline bool inner(const Oct &g, int i, int j, int k)
{
    return i >= 1 && i <= g.nx - 2 && j >= 1 && j <= g.ny - 2 && k >= 1 && k <= g.nz - 2;
}

// first weight slot of an octant (1, 2, 4: two slots; 3, 5, 6: four; 7: eight)
__host__ __device__ inline int wbase(int o)
{
    return o == 1 ? 0 : o == 2 ? 2 : o == 4 ? 4 : o == 3 ? 6 : o == 5 ? 10 : o == 6 ? 14 : 18;
}

// position of corner m (a subset of the odd bits o) among the corners of o
__host__ __device__ inline int wrank(int o, int m)
{
    int r = 0, s = 0;
    for (int d = 0; d < 3; ++d)
        if ((o >> d) & 1) {
            r |= ((m >> d) & 1) << s;
            ++s;
        }
    return r;
}

constexpr int NWSLOT = 26;

// Logical block of hardware block b in a grid of nb blocks (nb a multiple of
// 8).  Workgroups are dealt to the eight XCDs round-robin (b mod 8), each with
// its own L2; giving every XCD a contiguous range of logical blocks keeps the
// rows and planes that neighbouring blocks re-read in one L2.
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned nb)
{
    return (b & 7u) * (nb >> 3) + (b >> 3);
}

inline unsigned round8(unsigned n) { return (n + 7u) & ~7u; }

// sub-grid coordinates of thread t of an octant
__device__ inline void sub_coords(const Oct &g, long long t, int &a, int &b, int &c)
{
    a = (int)(t % g.px);
    const long long r = t / g.px;
    b = (int)(r % g.my);
    c = (int)(r / g.my);
}

// ---------------------------------------------------------------------------
// stencil access (setup kernels)
// ---------------------------------------------------------------------------
struct Sten {
    const double *p;   // npt 7: fields C, W, S, B; npt 27: C and 13 lower-half connections
    int npt;
    Oct g;
};

// all 27 entries A(p, p+d) of interior vertex (i,j,k), index (dz+1)*9+(dy+1)*3+(dx+1)
__device__ void load27(const Sten &s, int i, int j, int k, double e[27])
{
    const Oct &g = s.g;
    const long long v = vid(g, i, j, k);
    const long long F = g.field;
#pragma unroll
    for (int o = 0; o < 27; ++o) e[o] = 0.0;
    e[13] = s.p[v];
    if (s.npt == 7) {
        e[12] = -s.p[F + v];
        e[14] = -s.p[F + vid(g, i + 1, j, k)];
        e[10] = -s.p[2 * F + v];
        e[16] = -s.p[2 * F + vid(g, i, j + 1, k)];
        e[4] = -s.p[3 * F + v];
        e[22] = -s.p[3 * F + vid(g, i, j, k + 1)];
    } else {
#pragma unroll
        for (int o = 0; o < 13; ++o) {
            const int dx = o % 3 - 1, dy = (o / 3) % 3 - 1, dz = o / 9 - 1;
            e[o] = -s.p[(1 + o) * F + v];
            e[26 - o] = -s.p[(1 + o) * F + vid(g, i - dx, j - dy, k - dz)];
        }
    }
}

// ---------------------------------------------------------------------------
// layout conversion and finite volumes
// ---------------------------------------------------------------------------
// times scale; *tiny (or null) is set where an interior value is tiny_diag
__global__ void k3_to_oct(const double *nat, double *out, Oct g, int interior_only, double scale, int *tiny)
{
    const long long n = (long long)g.nx * g.ny * g.nz;
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int i = (int)(t % g.nx), j = (int)((t / g.nx) % g.ny), k = (int)(t / ((long long)g.nx * g.ny));
    const bool keep = !interior_only || inner(g, i, j, k);
    out[vid(g, i, j, k)] = keep ? scale * nat[t] : 0.0;
    if (tiny && hbmg::tiny_diag(nat[t]) && inner(g, i, j, k)) *tiny = 1;
}

__global__ void k3_from_oct(const double *in, double *nat, Oct g, double scale)
{
    const long long n = (long long)g.nx * g.ny * g.nz;
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int i = (int)(t % g.nx), j = (int)((t / g.nx) % g.ny), k = (int)(t / ((long long)g.nx * g.ny));
    nat[t] = inner(g, i, j, k) ? scale * in[vid(g, i, j, k)] : 0.0;
}

__device__ inline double cellv3(const double *D, int nx, int ny, int nz, int ci, int cj, int ck)
{
    if (ci < 0 || cj < 0 || ck < 0 || ci >= nx - 1 || cj >= ny - 1 || ck >= nz - 1) return 0.0;
    return D[((long long)ck * (ny - 1) + cj) * (nx - 1) + ci];
}

// connections of the edges ending at (i,j,k) from the west, south and below:
// the mean of the four cells around the edge (0 where undefined)
__device__ inline double fv_w(const double *D, int nx, int ny, int nz, int i, int j, int k)
{
    if (!(i >= 1 && j >= 1 && j <= ny - 2 && k >= 1 && k <= nz - 2)) return 0.0;
    return 0.25 * (cellv3(D, nx, ny, nz, i - 1, j - 1, k - 1) + cellv3(D, nx, ny, nz, i - 1, j, k - 1) +
                   cellv3(D, nx, ny, nz, i - 1, j - 1, k) + cellv3(D, nx, ny, nz, i - 1, j, k));
}
__device__ inline double fv_s(const double *D, int nx, int ny, int nz, int i, int j, int k)
{
    if (!(j >= 1 && i >= 1 && i <= nx - 2 && k >= 1 && k <= nz - 2)) return 0.0;
    return 0.25 * (cellv3(D, nx, ny, nz, i - 1, j - 1, k - 1) + cellv3(D, nx, ny, nz, i, j - 1, k - 1) +
                   cellv3(D, nx, ny, nz, i - 1, j - 1, k) + cellv3(D, nx, ny, nz, i, j - 1, k));
}
__device__ inline double fv_b(const double *D, int nx, int ny, int nz, int i, int j, int k)
{
    if (!(k >= 1 && i >= 1 && i <= nx - 2 && j >= 1 && j <= ny - 2)) return 0.0;
    return 0.25 * (cellv3(D, nx, ny, nz, i - 1, j - 1, k - 1) + cellv3(D, nx, ny, nz, i, j - 1, k - 1) +
                   cellv3(D, nx, ny, nz, i - 1, j, k - 1) + cellv3(D, nx, ny, nz, i, j, k - 1));
}

__global__ void k3_fv7(const double *D, int nx, int ny, int nz, double *planes)
{
    const long long n = (long long)nx * ny * nz;
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int i = (int)(t % nx), j = (int)((t / nx) % ny), k = (int)(t / ((long long)nx * ny));
    const double w = fv_w(D, nx, ny, nz, i, j, k);
    const double s = fv_s(D, nx, ny, nz, i, j, k);
    const double b = fv_b(D, nx, ny, nz, i, j, k);
    double c = 0.0;
    if (i >= 1 && i <= nx - 2 && j >= 1 && j <= ny - 2 && k >= 1 && k <= nz - 2)
        c = w + fv_w(D, nx, ny, nz, i + 1, j, k) + s + fv_s(D, nx, ny, nz, i, j + 1, k) + b +
            fv_b(D, nx, ny, nz, i, j, k + 1);
    planes[t] = c;
    planes[n + t] = w;
    planes[2 * n + t] = s;
    planes[3 * n + t] = b;
}

// ---------------------------------------------------------------------------
// interpolation weights (section 2; the 3D passes of section 3's cost count)
// ---------------------------------------------------------------------------
struct WArgs {
    Sten s;
    double *w;    // NWSLOT octant-sized slots of the fine level
    Oct c;        // coarse geometry
};

// acc[corner of p] += f * (interpolation row of the interior vertex q)
__device__ inline void add_row(const Oct &g, const double *w, int i, int j, int k, int qi, int qj, int qk, double f,
                               double acc[8])
{
    const int oq = oct_of(qi, qj, qk);
    const int bi = i >> 1, bj = j >> 1, bk = k >> 1;
    if (oq == 0) {
        const int m = ((qi >> 1) - bi) | (((qj >> 1) - bj) << 1) | (((qk >> 1) - bk) << 2);
        acc[m] += f;
        return;
    }
    const long long sq = sub_of(g, qi, qj, qk);
    for (int m = 0; m < 8; ++m) {
        if (m & ~oq) continue;
        const double wq = w[(wbase(oq) + wrank(oq, m)) * g.oct + sq];
        const int ci = (qi >> 1) + (m & 1) - bi, cj = (qj >> 1) + ((m >> 1) & 1) - bj,
                  ck = (qk >> 1) + (m >> 2) - bk;
        acc[ci | (cj << 1) | (ck << 2)] += f * wq;
    }
}

// PASS 1: line vertices (octants 1, 2, 4 by blockIdx.y); 2: face vertices
// (octants 6, 5, 3); 3: cell centres (octant 7).
template <int PASS>
__global__ __launch_bounds__(256) void k3_weights(WArgs a)
{
    const Oct g = a.s.g;
    const int y = blockIdx.y;
    const int o = PASS == 1 ? (1 << y) : PASS == 2 ? (7 ^ (1 << y)) : 7;
    const long long t = blockIdx.x * 256LL + threadIdx.x;
    if (t >= g.oct) return;
    int sa, sb, sc;
    sub_coords(g, t, sa, sb, sc);
    const int i = 2 * sa + (o & 1), j = 2 * sb + ((o >> 1) & 1), k = 2 * sc + (o >> 2);
    if (sa >= g.mx || !inner(g, i, j, k)) return;
    double e[27];
    load27(a.s, i, j, k, e);
    double acc[8];
    for (int m = 0; m < 8; ++m) acc[m] = 0.0;
    if (PASS == 1) {
        // the odd direction t1; the relation along the line after summing the
        // stencil over the two other directions
        const int t1 = y, o1 = t1 == 0 ? 1 : 0, o2 = t1 == 2 ? 1 : 2;
        double den = 0.0, am = 0.0, ap = 0.0;
        for (int u = -1; u <= 1; ++u)
            for (int v = -1; v <= 1; ++v) {
                int d[3];
                d[o1] = u;
                d[o2] = v;
                d[t1] = 0;
                den += e[(d[2] + 1) * 9 + (d[1] + 1) * 3 + (d[0] + 1)];
                d[t1] = -1;
                am += e[(d[2] + 1) * 9 + (d[1] + 1) * 3 + (d[0] + 1)];
                d[t1] = 1;
                ap += e[(d[2] + 1) * 9 + (d[1] + 1) * 3 + (d[0] + 1)];
            }
        acc[0] = -am / den;
        acc[o] = -ap / den;
    } else if (PASS == 2) {
        // the face normal n (the even direction): sum along it, then eliminate
        // the eight in-face neighbours
        const int n = y, o1 = n == 0 ? 1 : 0, o2 = n == 2 ? 1 : 2;
        double at[3][3];
        for (int s = 0; s < 3; ++s)
            for (int r = 0; r < 3; ++r) at[s][r] = 0.0;
        for (int s = -1; s <= 1; ++s)
            for (int r = -1; r <= 1; ++r)
                for (int m = -1; m <= 1; ++m) {
                    int d[3];
                    d[o1] = r;
                    d[o2] = s;
                    d[n] = m;
                    at[s + 1][r + 1] += e[(d[2] + 1) * 9 + (d[1] + 1) * 3 + (d[0] + 1)];
                }
        const double diag = at[1][1];
        for (int s = -1; s <= 1; ++s)
            for (int r = -1; r <= 1; ++r) {
                if (r == 0 && s == 0) continue;
                const double av = at[s + 1][r + 1];
                if (av == 0.0) continue;
                int d[3];
                d[o1] = r;
                d[o2] = s;
                d[n] = 0;
                const int qi = i + d[0], qj = j + d[1], qk = k + d[2];
                if (!inner(g, qi, qj, qk)) continue;
                add_row(g, a.w, i, j, k, qi, qj, qk, -av / diag, acc);
            }
    } else {
        const double diag = e[13];
        for (int q = 0; q < 27; ++q) {
            if (q == 13) continue;
            const double av = e[q];
            if (av == 0.0) continue;
            const int qi = i + q % 3 - 1, qj = j + (q / 3) % 3 - 1, qk = k + q / 9 - 1;
            if (!inner(g, qi, qj, qk)) continue;
            add_row(g, a.w, i, j, k, qi, qj, qk, -av / diag, acc);
        }
    }
    // no weight on boundary coarse vertices
    for (int m = 0; m < 8; ++m) {
        if (m & ~o) continue;
        const int I = (i >> 1) + (m & 1), J = (j >> 1) + ((m >> 1) & 1), K = (k >> 1) + (m >> 2);
        a.w[(wbase(o) + wrank(o, m)) * g.oct + t] = inner(a.c, I, J, K) ? acc[m] : 0.0;
    }
}

// ---------------------------------------------------------------------------
// Galerkin coarse operator A_c = P^T A P (section 2), one coarse vertex per
// thread: sum over its 27 fine support vertices p, their 27 couplings q, and
// the corners of q, keeping the lower half and the diagonal.
// ---------------------------------------------------------------------------
struct RArgs {
    Sten s;
    const double *w;
    Oct c;
    double *out;   // 14 coarse fields
};

__device__ inline double weight_on(const Oct &g, const double *w, int pi, int pj, int pk, int m)
{
    const int op = oct_of(pi, pj, pk);
    if (op == 0) return m == 0 ? 1.0 : 0.0;
    return w[(wbase(op) + wrank(op, m)) * g.oct + sub_of(g, pi, pj, pk)];
}

__global__ __launch_bounds__(256) void k3_rap(RArgs a)
{
    const Oct g = a.s.g, c = a.c;
    const long long t = blockIdx.x * 256LL + threadIdx.x;
    if (t >= c.field) return;
    const int oc = (int)(t / c.oct);
    int ca, cb, cc;
    sub_coords(c, t % c.oct, ca, cb, cc);
    const int I = 2 * ca + (oc & 1), J = 2 * cb + ((oc >> 1) & 1), K = 2 * cc + (oc >> 2);
    if (ca >= c.mx || !inner(c, I, J, K)) return;
    double acc[14];
    for (int o = 0; o < 14; ++o) acc[o] = 0.0;
    for (int ez = -1; ez <= 1; ++ez)
        for (int ey = -1; ey <= 1; ++ey)
            for (int ex = -1; ex <= 1; ++ex) {
                const int pi = 2 * I + ex, pj = 2 * J + ey, pk = 2 * K + ez;
                // p's corner that is I: the bit is set where e = -1
                const int mI = (ex == -1 ? 1 : 0) | (ey == -1 ? 2 : 0) | (ez == -1 ? 4 : 0);
                const double wp = weight_on(g, a.w, pi, pj, pk, mI);
                if (wp == 0.0) continue;
                double e[27];
                load27(a.s, pi, pj, pk, e);
                for (int f = 0; f < 27; ++f) {
                    const double av = e[f];
                    if (av == 0.0) continue;
                    const int qi = pi + f % 3 - 1, qj = pj + (f / 3) % 3 - 1, qk = pk + f / 9 - 1;
                    if (!inner(g, qi, qj, qk)) continue;
                    const int oq = oct_of(qi, qj, qk);
                    const double wa = wp * av;
                    for (int m = 0; m < 8; ++m) {
                        if (m & ~oq) continue;
                        const int dI = (qi >> 1) + (m & 1) - I, dJ = (qj >> 1) + ((m >> 1) & 1) - J,
                                  dK = (qk >> 1) + (m >> 2) - K;
                        const int lin = (dK + 1) * 9 + (dJ + 1) * 3 + (dI + 1);
                        if (lin > 13) continue;
                        acc[lin] += wa * weight_on(g, a.w, qi, qj, qk, m);
                    }
                }
            }
    a.out[t] = acc[13];
    for (int o = 0; o < 13; ++o) a.out[(1 + o) * c.field + t] = -acc[o];
}

// level operator in the plain layout: 27 entries per vertex, zero towards the boundary
__global__ void k3_stencil_out(Sten s, double *out, double scale)
{
    const Oct &g = s.g;
    const long long n = (long long)g.nx * g.ny * g.nz;
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int i = (int)(t % g.nx), j = (int)((t / g.nx) % g.ny), k = (int)(t / ((long long)g.nx * g.ny));
    double e[27];
    if (inner(g, i, j, k)) {
        load27(s, i, j, k, e);
        for (int o = 0; o < 27; ++o)
            if (o != 13 && !inner(g, i + o % 3 - 1, j + (o / 3) % 3 - 1, k + o / 9 - 1)) e[o] = 0.0;
    } else {
        for (int o = 0; o < 27; ++o) e[o] = 0.0;
    }
    for (int o = 0; o < 27; ++o) out[o * n + t] = scale * e[o];
}

__global__ void k3_interp_out(Oct g, const double *w, double *out)
{
    const long long n = (long long)g.nx * g.ny * g.nz;
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int i = (int)(t % g.nx), j = (int)((t / g.nx) % g.ny), k = (int)(t / ((long long)g.nx * g.ny));
    const bool in = inner(g, i, j, k);
    const int o = oct_of(i, j, k);
    for (int m = 0; m < 8; ++m) {
        double v = 0.0;
        if (in && !(m & ~o)) v = weight_on(g, w, i, j, k, m);
        out[m * n + t] = v;
    }
}

// ---------------------------------------------------------------------------
// solve phase
// ---------------------------------------------------------------------------
struct LArgs {
    Oct g;
    const double *st;  // stencil fields
    const double *b;
    double *x;
    double *r;         // residual out / in
    const double *w;   // weights (fine level)
    Oct c;             // coarse geometry
    const double *xc;
    double *bc;
    double *partials;
    int rescorr;
    double *xcz;       // restriction: the coarse iterate, cleared alongside (or null)
};

// index of the neighbour at (DX,DY,DZ) of thread t of octant O
template <int O, int DX, int DY, int DZ>
__device__ __forceinline__ long long nbr(const Oct &g, long long t)
{
    constexpr int ox = (O & 1) + DX, oy = ((O >> 1) & 1) + DY, oz = (O >> 2) + DZ;
    constexpr int on = (ox & 1) | ((oy & 1) << 1) | ((oz & 1) << 2);
    constexpr int sx = ox >> 1, sy = oy >> 1, sz = oz >> 1;
    return on * g.oct + t + sz * g.plane + sy * g.px + sx;
}

// The residual of row p, b_p - (A x)_p, as every kernel (grid-wide or
// collapsed) forms it: b_p - A_pp x_p, plus the sum of the terms of the planes
// above and below (off_plane, a chain of its own), then the terms of p's own
// plane (in_plane), each one fused multiply-add in a fixed order.  The
// relaxation adds it over A_pp to x_p.  Starting from the diagonal the partial
// sums shrink towards the residual, so their rounding does too.
template <int NPT, int O>
__device__ __forceinline__ double off_plane(const Oct &g, const double *st, const double *x, long long t)
{
    const long long F = g.field;
    const long long v = O * g.oct + t;
    double s = 0.0;
    if (NPT == 7) {
        const double *B = st + 3 * F;
        const long long zb = nbr<O, 0, 0, -1>(g, t), zt = nbr<O, 0, 0, 1>(g, t);
        s += B[v] * x[zb];
        s += B[zt] * x[zt];
    } else {
#define HB3_PAIR(o, dx, dy, dz)                                                                      \
    {                                                                                                \
        const long long qm = nbr<O, dx, dy, dz>(g, t), qp = nbr<O, -(dx), -(dy), -(dz)>(g, t);      \
        s += st[(1 + o) * F + v] * x[qm];                                                            \
        s += st[(1 + o) * F + qp] * x[qp];                                                           \
    }
        HB3_PAIR(0, -1, -1, -1) HB3_PAIR(1, 0, -1, -1) HB3_PAIR(2, 1, -1, -1)
        HB3_PAIR(3, -1, 0, -1) HB3_PAIR(4, 0, 0, -1) HB3_PAIR(5, 1, 0, -1)
        HB3_PAIR(6, -1, 1, -1) HB3_PAIR(7, 0, 1, -1) HB3_PAIR(8, 1, 1, -1)
#undef HB3_PAIR
    }
    return s;
}

// the in-plane connections of vertex t in the order in_plane takes them:
// west, east, south, north (7-point); south-west, north-east, south, north,
// south-east, north-west, west, east (27-point)
template <int NPT> struct InPlane { enum { n = NPT == 7 ? 4 : 8 }; };

template <int NPT, int O>
__device__ __forceinline__ void in_plane_coefs(const Oct &g, const double *st, long long t, double *k)
{
    const long long F = g.field;
    const long long v = O * g.oct + t;
    if (NPT == 7) {
        k[0] = st[F + v];
        k[1] = st[F + nbr<O, 1, 0, 0>(g, t)];
        k[2] = st[2 * F + v];
        k[3] = st[2 * F + nbr<O, 0, 1, 0>(g, t)];
    } else {
        k[0] = st[10 * F + v];
        k[1] = st[10 * F + nbr<O, 1, 1, 0>(g, t)];
        k[2] = st[11 * F + v];
        k[3] = st[11 * F + nbr<O, 0, 1, 0>(g, t)];
        k[4] = st[12 * F + v];
        k[5] = st[12 * F + nbr<O, -1, 1, 0>(g, t)];
        k[6] = st[13 * F + v];
        k[7] = st[13 * F + nbr<O, 1, 0, 0>(g, t)];
    }
}

// xn: the neighbours' values, as a function of their offset (dx, dy)
template <int NPT, typename X>
__device__ __forceinline__ double in_plane(const double *k, double s, X xn)
{
    if (NPT == 7) {
        s += k[0] * xn(-1, 0);
        s += k[1] * xn(1, 0);
        s += k[2] * xn(0, -1);
        s += k[3] * xn(0, 1);
    } else {
        s += k[0] * xn(-1, -1);
        s += k[1] * xn(1, 1);
        s += k[2] * xn(0, -1);
        s += k[3] * xn(0, 1);
        s += k[4] * xn(1, -1);
        s += k[5] * xn(-1, 1);
        s += k[6] * xn(-1, 0);
        s += k[7] * xn(1, 0);
    }
    return s;
}

template <int O>
__device__ __forceinline__ bool thread_vertex(const Oct &g, long long t, int &i, int &j, int &k)
{
    int a, b, c;
    sub_coords(g, t, a, b, c);
    i = 2 * a + (O & 1);
    j = 2 * b + ((O >> 1) & 1);
    k = 2 * c + (O >> 2);
    return a < g.mx && inner(g, i, j, k);
}

// ---------------------------------------------------------------------------
// relaxation by planes.  Colours 0..3 are the planes of even k, 4..7 those of
// odd k, and a plane couples only to the planes above and below, which are of
// the other parity.  So a sweep is two launches, the even planes (four colours
// in turn) and then the odd ones, and within a launch every plane is a
// two-dimensional four-colour relaxation whose terms of the neighbouring
// planes do not change: a thread loads its vertex's row of the operator and
// sums those terms before the first colour, the plane's iterate waits in LDS,
// and a colour costs four or eight LDS reads and a barrier.
//
// Small levels are bound by latency: a half sweep takes one memory round trip
// and four short phases, 6-7 us for a level of 9^3 to 65^3 where four launches
// of one colour each took 16-19 us.  All loads of a row go out before anything
// waits (a thread with the four rows of its cell kept them in batches: 15-20
// us).  Large ones are bound by memory: at 257^3 (7-point) a half sweep moves
// 622 MB in 125 us (5.0 TB/s; 543 MB if every value crossed once), at 129^3
// (27-point) 255 MB in 62 us.  Coefficients are plain loads: marked
// nontemporal, the connections that two rows of a tile share are fetched twice
// (257^3 102 -> 105-111 ms a solve).
//
// A workgroup owns tr rows of tc cells of a plane (a cell: the vertices of
// the plane's four octants with one sub-grid position).  What it needs from
// beyond its tile it relaxes itself: a chain of colours reaches one cell to
// the left, two to the right and one row up (its even-row colours only), and
// one cell and one row further down where the residual follows.  Rows and
// columns beyond that are read as they were before the half sweep, which is
// why the relaxed planes go to a second buffer.
// ---------------------------------------------------------------------------
struct Tile {
    int ncol, nrow, nk, kk0;   // cells and planes with interior vertices
    int tc, tr, ntx, nty;      // tiles of a plane
    int hx, hy;                // halo cells to the left, rows below
    int cw, rw;                // cells x rows relaxed
    int n01, n23;              // threads of an even-row and of an odd-row group
    unsigned ntiles;
};

struct PArgs {
    Oct g;
    const double *st, *b;
    const double *xs, *xo;     // the planes' own iterate, the other parity's
    double *xd;                // the relaxed planes
    double *r;
    const double *w;           // restriction
    Oct c;
    double *bc, *xcz;
    double *partials;
    Tile t;
};

// a thread's vertex: its row of the operator as loaded, then its off-plane sum
template <int NPT>
struct Row {
    enum { noff = NPT == 7 ? 2 : 18 };
    double b, off, d, y, k[InPlane<NPT>::n];   // y: 1 / d
    double oc[noff], ox[noff];
    bool in;
};

// every load of the row of vertex (i, j) of octant O, none of them waited
// for: at a vertex that is not interior they stay inside the fields, and are
// not used.  OFF: off-plane coefficients and iterate (1), coefficients alone (2)
template <int NPT, int O, bool ZC, int OFF>
__device__ __forceinline__ void load_row(const PArgs &a, int i, int j, long long t, Row<NPT> &R)
{
    R.in = i >= 1 && i <= a.g.nx - 2 && j >= 1 && j <= a.g.ny - 2;
    const long long F = a.g.field, v = O * a.g.oct + t;
    if (NPT == 7) {
        if (OFF || ZC) {
            R.oc[0] = a.st[3 * F + v];
            R.oc[1] = a.st[3 * F + nbr<O, 0, 0, 1>(a.g, t)];
        }
        if (OFF) {
            R.ox[0] = a.xo[nbr<O, 0, 0, -1>(a.g, t)];
            R.ox[1] = a.xo[nbr<O, 0, 0, 1>(a.g, t)];
        }
    } else if (OFF) {
#define HB3_PAIR(o, dx, dy)                                                                          \
    {                                                                                                \
        const long long qm = nbr<O, dx, dy, -1>(a.g, t), qp = nbr<O, -(dx), -(dy), 1>(a.g, t);       \
        R.oc[2 * o] = a.st[(1 + o) * F + v];                                                         \
        if (OFF == 1) R.ox[2 * o] = a.xo[qm];                                                        \
        R.oc[2 * o + 1] = a.st[(1 + o) * F + qp];                                                    \
        if (OFF == 1) R.ox[2 * o + 1] = a.xo[qp];                                                    \
    }
        HB3_PAIR(0, -1, -1) HB3_PAIR(1, 0, -1) HB3_PAIR(2, 1, -1)
        HB3_PAIR(3, -1, 0) HB3_PAIR(4, 0, 0) HB3_PAIR(5, 1, 0)
        HB3_PAIR(6, -1, 1) HB3_PAIR(7, 0, 1) HB3_PAIR(8, 1, 1)
#undef HB3_PAIR
    }
    in_plane_coefs<NPT, O>(a.g, a.st, t, R.k);
    if (!(NPT == 7 && ZC)) R.d = a.st[v];
    R.b = a.b[v];
}

// the off-plane sum (a chain in the order of the pairs), the diagonal's
// reciprocal (no colour phase waits for a division: 33^3 1208 -> 1189 us a solve,
// 129 x 97 x 65 7.26 -> 7.14 ms) and, where it is formed, the diagonal W_p + W_e + S_p + S_n + B_p + B_t (in this order the
// setup found it bitwise the stored one)
template <int NPT, bool ZC, bool OFF>
__device__ __forceinline__ void finish_row(Row<NPT> &R)
{
    R.off = 0.0;
    if (OFF) {
#pragma unroll
        for (int q = 0; q < Row<NPT>::noff; ++q) R.off += R.oc[q] * R.ox[q];
    }
    if (NPT == 7 && ZC) R.d = R.k[0] + R.k[1] + R.k[2] + R.k[3] + R.oc[0] + R.oc[1];
    R.y = 1.0 / R.d;
}

// the plane's iterate in LDS: one array per octant of the plane, rows lr0..,
// cells la0.. of the window
struct Window {
    double *x;
    int stride, size;
};

// value at (dx, dy) from the vertex of octant O (its plane's parity dropped) in cell `at`
template <int O>
__device__ __forceinline__ double win(const Window &w, int at, int dx, int dy)
{
    const int ox = (O & 1) + dx, oy = ((O >> 1) & 1) + dy;
    const int q = (ox & 1) | ((oy & 1) << 1);
    return w.x[q * w.size + at + (oy >> 1) * w.stride + (ox >> 1)];
}

template <int NPT, int Q>
__device__ __forceinline__ double row_resid(const Window &w, int at, const Row<NPT> &R)
{
    double s = R.b - R.d * w.x[Q * w.size + at];
    s += R.off;
    return in_plane<NPT>(R.k, s, [&](int dx, int dy) { return win<Q>(w, at, dx, dy); });
}

template <int NPT, int Q>
__device__ __forceinline__ void relax_colour(const Window &w, int at, const Row<NPT> &R)
{
    if (R.in) w.x[Q * w.size + at] += div_by(row_resid<NPT, Q>(w, at, R), R.d, R.y);
}

// the window's iterate into LDS: zero, or as stored
template <int PZ, bool ZERO>
__device__ __forceinline__ void fill_window(const PArgs &a, const Window &w, int la0, int lr0, int kk)
{
    for (int e = threadIdx.x; e < (ZERO ? 4 * w.size : w.size); e += blockDim.x) {
        if (ZERO) {
            w.x[e] = 0.0;
            continue;
        }
        const int row = e / w.stride, ca = la0 + e - row * w.stride, cr = lr0 + row;
        const double *x = a.xs + 4 * PZ * a.g.oct + (long long)kk * a.g.plane + (long long)cr * a.g.px + ca;
#pragma unroll
        for (int q = 0; q < 4; ++q) w.x[q * w.size + e] = x[q * a.g.oct];
    }
}

// fixed-order sum over the workgroup (up to 16 waves) into partials[blk]
__device__ __forceinline__ void block_partial(double sq, double *partials, unsigned blk)
{
    __shared__ double ws[16];
    for (int off = 32; off >= 1; off >>= 1) sq += __shfl_xor(sq, off, 64);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = ws[0];
        for (unsigned q = 1; q < (blockDim.x + 63) / 64; ++q) s += ws[q];
        partials[blk] = s;
    }
}

constexpr int PLANE_THREADS = 1024;

// a tile of a plane and a thread's part in it.  Threads come in groups by
// colour, padded to whole waves so that a wave's vertices are of one octant:
// 7-point levels have two (even rows: colours 0 and 1, both on one thread; odd
// rows: 2 and 3), 27-point levels, whose rows take 46 loads, one per colour.
template <int NPT>
struct Place {
    int kk, a0, a1, r0, r1;      // plane, owned cells and rows
    int la0, lr0, lr;            // window origin and rows
    Window w;
    int group, ca, cr, at;       // this thread's cell
    long long t;
    bool valid, own;

    __device__ __forceinline__ Place(const PArgs &a, unsigned lb, double *sx)
    {
        const Tile &T = a.t;
        const int tx = lb % T.ntx, ty = (lb / T.ntx) % T.nty;
        kk = T.kk0 + (int)(lb / (T.ntx * T.nty));
        a0 = tx * T.tc;
        a1 = min(a0 + T.tc, T.ncol);
        r0 = ty * T.tr;
        r1 = min(r0 + T.tr, T.nrow);
        const int ca0 = max(a0 - T.hx, 0), ca1 = min(a1 + 2, T.ncol), cr0 = max(r0 - T.hy, 0),
                  cr1 = min(r1 + 1, T.nrow);
        la0 = max(ca0 - 1, 0);
        lr0 = max(cr0 - 1, 0);
        lr = min(cr1, a.g.my - 1) - lr0 + 1;
        w.x = sx;
        w.stride = min(ca1, a.g.mx - 1) - la0 + 1;
        w.size = w.stride * lr;
        int e = threadIdx.x;
        if (NPT == 7) {
            group = e >= T.n01 ? 1 : 0;
            e -= group * T.n01;
        } else {
            group = e < T.n01 ? 0 : e < 2 * T.n01 ? 1 : e < 2 * T.n01 + T.n23 ? 2 : 3;
            e -= group < 2 ? group * T.n01 : 2 * T.n01 + (group - 2) * T.n23;
        }
        group = __builtin_amdgcn_readfirstlane(group);
        const bool odd = group >= (NPT == 7 ? 1 : 2);   // the row above the tile: even vertices only
        const int row = e / T.cw;
        ca = ca0 + e - row * T.cw;
        cr = cr0 + row;
        valid = ca < ca1 && cr < (odd ? r1 : cr1);
        own = valid && ca >= a0 && ca < a1 && cr >= r0 && cr < r1;
        // threads without a vertex load the tile's last
        ca = min(ca, ca1 - 1);
        cr = min(cr, (odd ? r1 : cr1) - 1);
        at = (cr - lr0) * w.stride + ca - la0;
        t = (long long)kk * a.g.plane + (long long)cr * a.g.px + ca;
    }
};

template <int NPT> struct Pts { enum { n = NPT == 7 ? 2 : 1 }; };   // vertices of a thread

template <int NPT, int PZ, bool ZC, bool OFF>
__device__ __forceinline__ void load_rows(const PArgs &a, const Place<NPT> &P, Row<NPT> *R)
{
    const int i = 2 * P.ca, j = 2 * P.cr;
    if (NPT == 7) {
        if (P.group == 0) {
            load_row<NPT, 4 * PZ + 0, ZC, OFF>(a, i, j, P.t, R[0]);
            load_row<NPT, 4 * PZ + 1, ZC, OFF>(a, i + 1, j, P.t, R[Pts<NPT>::n - 1]);
        } else {
            load_row<NPT, 4 * PZ + 2, ZC, OFF>(a, i, j + 1, P.t, R[0]);
            load_row<NPT, 4 * PZ + 3, ZC, OFF>(a, i + 1, j + 1, P.t, R[Pts<NPT>::n - 1]);
        }
    } else {
        if (P.group == 0) load_row<NPT, 4 * PZ + 0, ZC, OFF>(a, i, j, P.t, R[0]);
        else if (P.group == 1) load_row<NPT, 4 * PZ + 1, ZC, OFF>(a, i + 1, j, P.t, R[0]);
        else if (P.group == 2) load_row<NPT, 4 * PZ + 2, ZC, OFF>(a, i, j + 1, P.t, R[0]);
        else load_row<NPT, 4 * PZ + 3, ZC, OFF>(a, i + 1, j + 1, P.t, R[0]);
    }
#pragma unroll
    for (int q = 0; q < Pts<NPT>::n; ++q) R[q].in = R[q].in && P.valid;
}

// f(colour constant, row) for this thread's vertices
template <int NPT, typename Fn>
__device__ __forceinline__ void each_vertex(const Place<NPT> &P, const Row<NPT> *R, Fn f)
{
    if (NPT == 7) {
        if (P.group == 0) {
            f(std::integral_constant<int, 0>{}, R[0]);
            f(std::integral_constant<int, 1>{}, R[Pts<NPT>::n - 1]);
        } else {
            f(std::integral_constant<int, 2>{}, R[0]);
            f(std::integral_constant<int, 3>{}, R[Pts<NPT>::n - 1]);
        }
    } else {
        if (P.group == 0) f(std::integral_constant<int, 0>{}, R[0]);
        else if (P.group == 1) f(std::integral_constant<int, 1>{}, R[0]);
        else if (P.group == 2) f(std::integral_constant<int, 2>{}, R[0]);
        else f(std::integral_constant<int, 3>{}, R[0]);
    }
}

template <int NPT, int Q>
__device__ __forceinline__ void colour_phase(const Place<NPT> &P, const Row<NPT> *R)
{
    constexpr int grp = NPT == 7 ? Q >> 1 : Q, q = NPT == 7 ? Q & 1 : 0;
    if (P.group == grp) relax_colour<NPT, Q>(P.w, P.at, R[q]);
}

// squares of the residual at this thread's own vertices
template <int NPT>
__device__ __forceinline__ double squares(const Place<NPT> &P, const Row<NPT> *R)
{
    double sq = 0.0;
    if (P.own)
        each_vertex<NPT>(P, R, [&](auto c, const Row<NPT> &r) {
            constexpr int Q = decltype(c)::value;
            if (!r.in) return;
            const double q = row_resid<NPT, Q>(P.w, P.at, r);
            sq += q * q;
        });
    return sq;
}

// Half a sweep: colours 4 PZ .. 4 PZ + 3 on the planes of parity PZ.
// ZERO: the sweep starts from x = 0 (the even planes then read no iterate and
// no coefficient towards other planes).  RES: 1 stores the residual the relaxed
// planes end with, 2 sums its squares (both only right for PZ = 1, the end of
// the sweep); 3 sums the squares of the residual they start with.
template <int NPT, int PZ, bool ZC, bool ZERO, int RES>
__global__ __launch_bounds__(PLANE_THREADS) void k3_plane(PArgs a)
{
    extern __shared__ double sx[];
    const unsigned lb = xcd_block(blockIdx.x, gridDim.x);
    if (lb >= a.t.ntiles) {
        if (RES >= 2 && threadIdx.x == 0) a.partials[lb] = 0.0;
        return;
    }
    const Place<NPT> P(a, lb, sx);
    constexpr bool OFF = !(ZERO && PZ == 0);
    Row<NPT> R[Pts<NPT>::n];
    load_rows<NPT, PZ, ZC, OFF>(a, P, R);
    fill_window<PZ, ZERO>(a, P.w, P.la0, P.lr0, P.kk);
#pragma unroll
    for (int q = 0; q < Pts<NPT>::n; ++q) finish_row<NPT, ZC, OFF>(R[q]);
    __syncthreads();
    double sq = 0.0;
    if (RES == 3) {
        sq = squares(P, R);
        __syncthreads();
    }
    colour_phase<NPT, 0>(P, R);
    __syncthreads();
    colour_phase<NPT, 1>(P, R);
    __syncthreads();
    colour_phase<NPT, 2>(P, R);
    __syncthreads();
    colour_phase<NPT, 3>(P, R);
    if (RES == 1 || RES == 2) __syncthreads();
    if (P.own) {
        const long long v = 4 * PZ * a.g.oct + P.t;
        each_vertex<NPT>(P, R, [&](auto c, const Row<NPT> &r) {
            constexpr int Q = decltype(c)::value;
            if (!r.in) return;
            a.xd[v + Q * a.g.oct] = P.w.x[Q * P.w.size + P.at];
            if (RES == 1) a.r[v + Q * a.g.oct] = row_resid<NPT, Q>(P.w, P.at, r);
        });
    }
    if (RES == 2) sq = squares(P, R);
    if (RES >= 2) block_partial(sq, a.partials, lb);
}

// A whole sweep of a 27-point level whose planes have at most 64 cells, nz odd: a
// workgroup relaxes one odd plane (z = 2 kk + 1) and, for itself, the even planes
// below and above it, four waves (a colour each, a cell per lane) to a plane; the
// odd plane's off-plane sum then comes from LDS.  It stores the odd plane and the
// even one below.  Such a level's half sweeps are launch and memory latency: at
// 17^3 two of them take 9-11 us, this 5.7-8.3 (33^3 968 -> 908 us a solve, 129 x 97
// x 65 5.89 -> 5.75 ms).  The same terms in the same order, so the same bits.
template <bool ZERO, int RES>
__global__ __launch_bounds__(768) void k3_sweep(PArgs a)
{
    extern __shared__ double sx[];
    const int pl = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);   // even below, even above, odd
    const int grp = __builtin_amdgcn_readfirstlane(((int)threadIdx.x >> 6) & 3), lane = threadIdx.x & 63;
    const Oct &g = a.g;
    const int kk = blockIdx.x, pk = pl == 1 ? kk + 1 : kk;
    const bool zin = pl == 2 || (pl == 0 ? kk >= 1 : 2 * kk + 2 <= g.nz - 2);
    const int ncol = (g.nx - 2) / 2 + 1, nrow = (g.ny - 2) / 2 + 1;
    const int size = g.mx * g.my;
    const Window w{sx + pl * 4 * size, g.mx, size};
    const bool valid = zin && lane < ncol * nrow;
    const int c = valid ? lane : 0, cr = c / ncol, ca = c - cr * ncol, at = cr * g.mx + ca;
    const long long t = (long long)pk * g.plane + (long long)cr * g.px + ca;
    Row<27> R;
    R.in = false;
    if (zin) {
        const int i = 2 * ca + (grp & 1), j = 2 * cr + (grp >> 1);
        if (pl < 2) {
            constexpr int OFF = ZERO ? 0 : 1;
            if (grp == 0) load_row<27, 0, false, OFF>(a, i, j, t, R);
            else if (grp == 1) load_row<27, 1, false, OFF>(a, i, j, t, R);
            else if (grp == 2) load_row<27, 2, false, OFF>(a, i, j, t, R);
            else load_row<27, 3, false, OFF>(a, i, j, t, R);
        } else {
            if (grp == 0) load_row<27, 4, false, 2>(a, i, j, t, R);
            else if (grp == 1) load_row<27, 5, false, 2>(a, i, j, t, R);
            else if (grp == 2) load_row<27, 6, false, 2>(a, i, j, t, R);
            else load_row<27, 7, false, 2>(a, i, j, t, R);
        }
    }
    R.in = R.in && valid;
    for (int e = threadIdx.x & 255; e < size; e += 256) {
        const int row = e / g.mx, col = e - row * g.mx;
        const double *x = a.xs + (pl == 2 ? 4 : 0) * g.oct + (long long)pk * g.plane + (long long)row * g.px + col;
#pragma unroll
        for (int q = 0; q < 4; ++q) w.x[q * size + e] = ZERO || !zin ? 0.0 : x[q * g.oct];
    }
    if (zin) {
        if (pl < 2) finish_row<27, false, !ZERO>(R);
        else R.y = 1.0 / R.d;
    }
    __syncthreads();
    auto colours = [&](bool mine) {
        if (mine && grp == 0) relax_colour<27, 0>(w, at, R);
        __syncthreads();
        if (mine && grp == 1) relax_colour<27, 1>(w, at, R);
        __syncthreads();
        if (mine && grp == 2) relax_colour<27, 2>(w, at, R);
        __syncthreads();
        if (mine && grp == 3) relax_colour<27, 3>(w, at, R);
        __syncthreads();
    };
    colours(pl < 2);
    if (pl == 2) {
        const Window lo{sx, g.mx, size}, hi{sx + 4 * size, g.mx, size};
        auto off = [&](auto q) {
            constexpr int Q = decltype(q)::value;
            double s = 0.0;
            if (R.in) {
#pragma unroll
                for (int o = 0; o < 9; ++o) {
                    s += R.oc[2 * o] * win<Q>(lo, at, o % 3 - 1, o / 3 - 1);
                    s += R.oc[2 * o + 1] * win<Q>(hi, at, 1 - o % 3, 1 - o / 3);
                }
            }
            R.off = s;
        };
        if (grp == 0) off(std::integral_constant<int, 0>{});
        else if (grp == 1) off(std::integral_constant<int, 1>{});
        else if (grp == 2) off(std::integral_constant<int, 2>{});
        else off(std::integral_constant<int, 3>{});
    }
    colours(pl == 2);
    if (!R.in || pl == 1) return;
    const long long v = ((pl == 2 ? 4 : 0) + grp) * g.oct + t;
    a.xd[v] = w.x[grp * size + at];
    if (RES == 1 && pl == 2) {
        if (grp == 0) a.r[v] = row_resid<27, 0>(w, at, R);
        else if (grp == 1) a.r[v] = row_resid<27, 1>(w, at, R);
        else if (grp == 2) a.r[v] = row_resid<27, 2>(w, at, R);
        else a.r[v] = row_resid<27, 3>(w, at, R);
    }
}

// Residual on the planes of parity PZ with the same tiles.  NORM: its squares'
// block sums, over the same threads and in the same order as k3_plane does
// with RES 2 (PZ = 1) and 3 (PZ = 0).
// Otherwise (PZ = 0): with the odd planes' residual in a.r already, the
// restriction as well: coarse vertex (I, J, K) sits in cell (I, J) of the even
// plane K and gathers this plane's residual from LDS (a halo cell to the left
// and a halo row below) and its neighbours' from memory, so the even planes'
// is written only for the interpolation's r/C and never read back here.
template <int NPT, int PZ, bool ZC, bool NORM>
__global__ __launch_bounds__(PLANE_THREADS) void k3_plane_resid(PArgs a)
{
    extern __shared__ double sx[];
    const unsigned lb = xcd_block(blockIdx.x, gridDim.x);
    if (lb >= a.t.ntiles) {
        if (NORM && threadIdx.x == 0) a.partials[lb] = 0.0;
        return;
    }
    const Place<NPT> P(a, lb, sx);
    Row<NPT> R[Pts<NPT>::n];
    load_rows<NPT, PZ, ZC, true>(a, P, R);
    fill_window<PZ, false>(a, P.w, P.la0, P.lr0, P.kk);
#pragma unroll
    for (int q = 0; q < Pts<NPT>::n; ++q) finish_row<NPT, ZC, true>(R[q]);
    __syncthreads();
    if (NORM) {
        block_partial(squares(P, R), a.partials, lb);
        return;
    }
    const long long v = 4 * PZ * a.g.oct + P.t;
    double rv[Pts<NPT>::n];
    each_vertex<NPT>(P, R, [&](auto c, const Row<NPT> &r) {
        constexpr int Q = decltype(c)::value;
        const double q = r.in ? row_resid<NPT, Q>(P.w, P.at, r) : 0.0;
        if (Q != 0 && P.own && r.in) a.r[v + Q * a.g.oct] = q;
        rv[(NPT == 7 ? Q & 1 : 0)] = q;
    });
    __syncthreads();   // every read of the iterate is done: its window takes the residual
    each_vertex<NPT>(P, R, [&](auto c, const Row<NPT> &) {
        constexpr int Q = decltype(c)::value;
        if (P.valid) P.w.x[Q * P.w.size + P.at] = rv[(NPT == 7 ? Q & 1 : 0)];
    });
    __syncthreads();
    if (P.group != 0 || !P.own || !inner(a.c, P.ca, P.cr, P.kk)) return;
    const Oct &g = a.g;
    double s = 0.0;
#pragma unroll
    for (int ez = -1; ez <= 1; ++ez)
#pragma unroll
        for (int ey = -1; ey <= 1; ++ey)
#pragma unroll
            for (int ex = -1; ex <= 1; ++ex) {
                const int pi = 2 * P.ca + ex, pj = 2 * P.cr + ey, pk = 2 * P.kk + ez;
                const int mI = (ex == -1 ? 1 : 0) | (ey == -1 ? 2 : 0) | (ez == -1 ? 4 : 0);
                const double q = ez == 0 ? win<0>(P.w, P.at, ex, ey) : a.r[vid(g, pi, pj, pk)];
                s += weight_on(g, a.w, pi, pj, pk, mI) * q;
            }
    const long long vc = vid(a.c, P.ca, P.cr, P.kk);
    a.bc[vc] = s;
    if (a.xcz) a.xcz[vc] = 0.0;
}

// residual r = b - A x of a whole level; blocks interleave the octants
// (octant = block mod 8), so that the eight octants of one region run together
// and share their neighbours in L2
template <int NPT, int O>
__device__ __forceinline__ void resid_at(const LArgs &a, long long t)
{
    int i, j, k;
    const Oct &g = a.g;
    if (!thread_vertex<O>(g, t, i, j, k)) {
        a.r[O * g.oct + t] = 0.0;
        return;
    }
    const long long v = O * g.oct + t;
    double kc[InPlane<NPT>::n];
    in_plane_coefs<NPT, O>(g, a.st, t, kc);
    double s = a.b[v] - a.st[v] * a.x[v];
    s += off_plane<NPT, O>(g, a.st, a.x, t);
    a.r[v] = in_plane<NPT>(kc, s, [&](int dx, int dy) {
        const int ox = (O & 1) + dx, oy = ((O >> 1) & 1) + dy;
        const long long q = ((ox & 1) | ((oy & 1) << 1) | (O & 4)) * g.oct + t;
        return a.x[q + (oy >> 1) * g.px + (ox >> 1)];
    });
}

template <int NPT>
__global__ __launch_bounds__(256) void k3_resid(LArgs a)
{
    const unsigned lb = xcd_block(blockIdx.x, gridDim.x);
    const long long t = (lb >> 3) * 256LL + threadIdx.x;
    if (t >= a.g.oct) return;
    switch (lb & 7) {
    case 0: resid_at<NPT, 0>(a, t); break;
    case 1: resid_at<NPT, 1>(a, t); break;
    case 2: resid_at<NPT, 2>(a, t); break;
    case 3: resid_at<NPT, 3>(a, t); break;
    case 4: resid_at<NPT, 4>(a, t); break;
    case 5: resid_at<NPT, 5>(a, t); break;
    case 6: resid_at<NPT, 6>(a, t); break;
    default: resid_at<NPT, 7>(a, t); break;
    }
}

// ZC check of a 7-point level: clears *flag unless every interior vertex's
// diagonal is bitwise W_p + W_e + S_p + S_n + B_p + B_t (finite volumes of
// pure diffusion build it so); blocks interleave the octants
template <int O>
__device__ __forceinline__ bool zexc7_at(const Oct &g, const double *st, long long t)
{
    int i, j, k;
    if (!thread_vertex<O>(g, t, i, j, k)) return true;
    const long long F = g.field, v = O * g.oct + t;
    const double *C = st, *W = st + F, *S = st + 2 * F, *B = st + 3 * F;
    const long long xe = nbr<O, 1, 0, 0>(g, t), yn = nbr<O, 0, 1, 0>(g, t), zt = nbr<O, 0, 0, 1>(g, t);
    return C[v] == W[v] + W[xe] + S[v] + S[yn] + B[v] + B[zt];
}

__global__ __launch_bounds__(256) void k3_zero_excess7(Oct g, const double *st, int *flag)
{
    const unsigned lb = blockIdx.x;
    const long long t = (lb >> 3) * 256LL + threadIdx.x;
    if (t >= g.oct) return;
    bool ok = true;
    switch (lb & 7) {
    case 0: ok = zexc7_at<0>(g, st, t); break;
    case 1: ok = zexc7_at<1>(g, st, t); break;
    case 2: ok = zexc7_at<2>(g, st, t); break;
    case 3: ok = zexc7_at<3>(g, st, t); break;
    case 4: ok = zexc7_at<4>(g, st, t); break;
    case 5: ok = zexc7_at<5>(g, st, t); break;
    case 6: ok = zexc7_at<6>(g, st, t); break;
    default: ok = zexc7_at<7>(g, st, t); break;
    }
    if (!ok) atomicAnd(flag, 0);
}

__global__ void k3_set_int(int *p, int v) { *p = v; }

// sum of squares of a field's interior entries (the norm of b), block sums
__global__ __launch_bounds__(256) void k3_sumsq(Oct g, const double *f, double *partials)
{
    const long long t = blockIdx.x * 256LL + threadIdx.x;
    double sq = 0.0;
    if (t < g.field) {
        const int o = (int)(t / g.oct);
        int a, b, c;
        sub_coords(g, t % g.oct, a, b, c);
        const int i = 2 * a + (o & 1), j = 2 * b + ((o >> 1) & 1), k = 2 * c + (o >> 2);
        if (a < g.mx && inner(g, i, j, k)) sq = f[t] * f[t];
    }
    for (int off = 32; off >= 1; off >>= 1) sq += __shfl_xor(sq, off, 64);
    __shared__ double ws[4];
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) partials[blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
}

// zero a field (a kernel, not a memset node, so that it can sit in a captured graph)
__global__ __launch_bounds__(256) void k3_fill0(double *p, long long n)
{
    for (long long t = blockIdx.x * 256LL + threadIdx.x; t < n; t += (long long)gridDim.x * 256) p[t] = 0.0;
}

// sum of partials [lo, hi) over a workgroup of 256; the result is thread 0's
__device__ __forceinline__ double sum_range(const double *partials, long long lo, long long hi)
{
    double s = 0.0;
    for (long long t = lo + threadIdx.x; t < hi; t += 256) s += partials[t];
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    __shared__ double ws[4];
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    return ws[0] + ws[1] + ws[2] + ws[3];
}

// block b: out[b] = sum of partials [b*chunk, min(n, (b+1)*chunk))
__global__ __launch_bounds__(256) void k3_reduce(const double *partials, long long n, long long chunk, double *out)
{
    const long long lo = blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    const double s = sum_range(partials, lo, hi);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// The sum of n partials to the host-mapped slot {sum, tag} the host polls.  The
// tag is `set` (it starts a solve) or the last one plus 1: a captured launch has
// no argument to carry it.  A copy to the host and a wait for the stream took
// 10 us a cycle more than the poll.
__global__ __launch_bounds__(256) void k3_sum_out(const double *partials, long long n, double *tag, double set,
                                                  double *slot)
{
    const double s = sum_range(partials, 0, n);
    if (threadIdx.x != 0) return;
    const double t = set != 0.0 ? set : *tag + 1.0;
    *tag = t;
    volatile double *v = slot;
    v[0] = s;
    __threadfence_system();
    v[1] = t;
}

// b_c = P^T r: each coarse vertex gathers its 27 fine support vertices
__global__ __launch_bounds__(256) void k3_restrict(LArgs a)
{
    const Oct g = a.g, c = a.c;
    // blocks interleave the coarse octants: neighbouring coarse vertices,
    // which share fine support vertices, run together
    const unsigned lb = xcd_block(blockIdx.x, gridDim.x);
    const int oc = lb & 7;
    const long long ts = (lb >> 3) * 256LL + threadIdx.x;
    if (ts >= c.oct) return;
    const long long t = oc * c.oct + ts;
    int ca, cb, cc;
    sub_coords(c, ts, ca, cb, cc);
    const int I = 2 * ca + (oc & 1), J = 2 * cb + ((oc >> 1) & 1), K = 2 * cc + (oc >> 2);
    // the coarse level's iterate starts at zero (every entry, boundary included)
    if (a.xcz) a.xcz[t] = 0.0;
    if (ca >= c.mx || !inner(c, I, J, K)) {
        a.bc[t] = 0.0;
        return;
    }
    double s = 0.0;
    // unrolled, the fine octant of every support vertex is a constant and the
    // 54 loads can go out together
#pragma unroll
    for (int ez = -1; ez <= 1; ++ez)
#pragma unroll
        for (int ey = -1; ey <= 1; ++ey)
#pragma unroll
            for (int ex = -1; ex <= 1; ++ex) {
                const int pi = 2 * I + ex, pj = 2 * J + ey, pk = 2 * K + ez;
                const int mI = (ex == -1 ? 1 : 0) | (ey == -1 ? 2 : 0) | (ez == -1 ? 4 : 0);
                s += weight_on(g, a.w, pi, pj, pk, mI) * a.r[vid(g, pi, pj, pk)];
            }
    a.bc[t] = s;
}

// x += P x_c (+ r/C at vertices that are not coarse points); blockIdx.y = octant
template <int NPT, int O>
__device__ __forceinline__ void interp_at(const LArgs &a, long long t)
{
    int i, j, k;
    if (!thread_vertex<O>(a.g, t, i, j, k)) return;
    const Oct &g = a.g, &c = a.c;
    const long long v = O * g.oct + t;
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        if (m & ~O) continue;
        const double w = O == 0 ? 1.0 : a.w[(wbase(O) + wrank(O, m)) * g.oct + t];
        s += w * a.xc[vid(c, (i >> 1) + (m & 1), (j >> 1) + ((m >> 1) & 1), (k >> 1) + (m >> 2))];
    }
    double xv = a.x[v] + s;
    if (O != 0 && a.rescorr) xv += a.r[v] / a.st[v];
    a.x[v] = xv;
}

template <int NPT>
__global__ __launch_bounds__(256) void k3_interp(LArgs a)
{
    const long long t = xcd_block(blockIdx.x, gridDim.x) * 256LL + threadIdx.x;
    if (t >= a.g.oct) return;
    switch (blockIdx.y) {
    case 0: interp_at<NPT, 0>(a, t); break;
    case 1: interp_at<NPT, 1>(a, t); break;
    case 2: interp_at<NPT, 2>(a, t); break;
    case 3: interp_at<NPT, 3>(a, t); break;
    case 4: interp_at<NPT, 4>(a, t); break;
    case 5: interp_at<NPT, 5>(a, t); break;
    case 6: interp_at<NPT, 6>(a, t); break;
    default: interp_at<NPT, 7>(a, t); break;
    }
}

// ---------------------------------------------------------------------------
// collapsed levels: levels 0..top in one persistent workgroup (the one-GPU
// form of the paper's coarse-grid redistribution).  Every phase does the
// arithmetic of the grid-wide kernels in the same expression order, so the
// iteration does not depend on the collapse level.
// ---------------------------------------------------------------------------
constexpr int MAXC3 = 8;
constexpr int CWG3 = 512;

struct CLev {
    Oct g;
    int npt;
    const double *st;
    const double *w;
    double *x, *b, *r;
};

struct CArgs {
    CLev lv[MAXC3];
    int top;
    const double *chol;
    const long long *cidx;
    int nc;
    int nu1, nu2, rescorr;
};

// collapsed levels are small (the host caps l* so that every plane offset of a
// collapsed level fits in 32 bits): 32-bit index arithmetic throughout, which
// keeps the runtime-octant stencil within the workgroup's register budget
__device__ __forceinline__ int nbr_rt(const Oct &g, int o, int t, int dx, int dy, int dz)
{
    const int ox = (o & 1) + dx, oy = ((o >> 1) & 1) + dy, oz = (o >> 2) + dz;
    const int on = (ox & 1) | ((oy & 1) << 1) | ((oz & 1) << 2);
    return on * (int)g.oct + t + (oz >> 1) * (int)g.plane + (oy >> 1) * g.px + (ox >> 1);
}

// the residual of a row with the octant at run time (same terms, same order)
__device__ __forceinline__ double row_rt(const CLev &L, int o, int t)
{
    const Oct &g = L.g;
    const int F = (int)g.field;
    const int v = o * (int)g.oct + t;
    const double *st = L.st, *x = L.x;
    double s = L.b[v] - st[v] * x[v], off = 0.0;
    if (L.npt == 7) {
        const double *W = st + F, *S = st + 2 * F, *B = st + 3 * F;
        const int xw = nbr_rt(g, o, t, -1, 0, 0), xe = nbr_rt(g, o, t, 1, 0, 0);
        const int ys = nbr_rt(g, o, t, 0, -1, 0), yn = nbr_rt(g, o, t, 0, 1, 0);
        const int zb = nbr_rt(g, o, t, 0, 0, -1), zt = nbr_rt(g, o, t, 0, 0, 1);
        off += B[v] * x[zb];
        off += B[zt] * x[zt];
        s += off;
        s += W[v] * x[xw];
        s += W[xe] * x[xe];
        s += S[v] * x[ys];
        s += S[yn] * x[yn];
        return s;
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int dx = q % 3 - 1, dy = q / 3 - 1;
        const int qm = nbr_rt(g, o, t, dx, dy, -1), qp = nbr_rt(g, o, t, -dx, -dy, 1);
        off += st[(1 + q) * F + v] * x[qm];
        off += st[(1 + q) * F + qp] * x[qp];
    }
    s += off;
#pragma unroll
    for (int q = 9; q < 13; ++q) {
        const int dx = q % 3 - 1, dy = (q / 3) % 3 - 1;
        const int qm = nbr_rt(g, o, t, dx, dy, 0), qp = nbr_rt(g, o, t, -dx, -dy, 0);
        s += st[(1 + q) * F + v] * x[qm];
        s += st[(1 + q) * F + qp] * x[qp];
    }
    return s;
}

// collapsed levels are small (fields < 2^31 entries): 32-bit index arithmetic
__device__ __forceinline__ void sub_coords32(const Oct &g, int t, int &a, int &b, int &c)
{
    a = t % g.px;
    const int r = t / g.px;
    b = r % g.my;
    c = r / g.my;
}

__device__ __forceinline__ bool vertex_rt(const Oct &g, int o, int t, int &i, int &j, int &k)
{
    int a, b, c;
    sub_coords32(g, t, a, b, c);
    i = 2 * a + (o & 1);
    j = 2 * b + ((o >> 1) & 1);
    k = 2 * c + (o >> 2);
    return a < g.mx && inner(g, i, j, k);
}

__device__ __forceinline__ void wg_relax(const CLev &L, int sweeps)
{
    for (int it = 0; it < sweeps; ++it)
        for (int o = 0; o < 8; ++o) {
            for (int t = threadIdx.x; t < (int)L.g.oct; t += CWG3) {
                int i, j, k;
                if (!vertex_rt(L.g, o, t, i, j, k)) continue;
                const int v = o * (int)L.g.oct + t;
                L.x[v] += row_rt(L, o, t) / L.st[v];
            }
            __syncthreads();
        }
}

__device__ __forceinline__ void wg_residual(const CLev &L)
{
    const int oct = (int)L.g.oct;
    for (int u = threadIdx.x; u < (int)L.g.field; u += CWG3) {
        const int o = u / oct;
        const int t = u - o * oct;
        int i, j, k;
        if (!vertex_rt(L.g, o, t, i, j, k)) {
            L.r[u] = 0.0;
            continue;
        }
        L.r[u] = row_rt(L, o, t);
    }
    __syncthreads();
}

__device__ __forceinline__ void wg_restrict(const CLev &F, const CLev &C)
{
    const Oct &g = F.g, &c = C.g;
    const int coct = (int)c.oct;
    for (int u = threadIdx.x; u < (int)c.field; u += CWG3) {
        const int oc = u / coct;
        int ca, cb, cc;
        sub_coords32(c, u - oc * coct, ca, cb, cc);
        const int I = 2 * ca + (oc & 1), J = 2 * cb + ((oc >> 1) & 1), K = 2 * cc + (oc >> 2);
        if (ca >= c.mx || !inner(c, I, J, K)) {
            C.b[u] = 0.0;
            continue;
        }
        double s = 0.0;
        for (int ez = -1; ez <= 1; ++ez)
            for (int ey = -1; ey <= 1; ++ey)
                for (int ex = -1; ex <= 1; ++ex) {
                    const int pi = 2 * I + ex, pj = 2 * J + ey, pk = 2 * K + ez;
                    const int mI = (ex == -1 ? 1 : 0) | (ey == -1 ? 2 : 0) | (ez == -1 ? 4 : 0);
                    s += weight_on(g, F.w, pi, pj, pk, mI) * F.r[vid(g, pi, pj, pk)];
                }
        C.b[u] = s;
    }
    // the coarse iterate starts at zero
    for (long long u = threadIdx.x; u < c.field; u += CWG3) C.x[u] = 0.0;
    __syncthreads();
}

__device__ __forceinline__ void wg_interp(const CLev &F, const CLev &C, int rescorr)
{
    const Oct &g = F.g, &c = C.g;
    const int oct = (int)g.oct;
    for (int u = threadIdx.x; u < (int)g.field; u += CWG3) {
        const int o = u / oct;
        const int t = u - o * oct;
        int i, j, k;
        if (!vertex_rt(g, o, t, i, j, k)) continue;
        double s = 0.0;
        for (int m = 0; m < 8; ++m) {
            if (m & ~o) continue;
            const double w = o == 0 ? 1.0 : F.w[(wbase(o) + wrank(o, m)) * g.oct + t];
            s += w * C.x[vid(c, (i >> 1) + (m & 1), (j >> 1) + ((m >> 1) & 1), (k >> 1) + (m >> 2))];
        }
        double xv = F.x[u] + s;
        if (o != 0 && rescorr) xv += F.r[u] / F.st[u];
        F.x[u] = xv;
    }
    __syncthreads();
}

__device__ void wg_coarse(const CArgs &a, double *y)
{
    const int n = a.nc;
    const double *Lf = a.chol;
    for (int r = threadIdx.x; r < n; r += CWG3) y[r] = a.lv[0].b[a.cidx[r]];
    __syncthreads();
    for (int k = 0; k < n; ++k) {
        const double yk = y[k] / Lf[(long long)k * n + k];
        __syncthreads();
        if (threadIdx.x == 0) y[k] = yk;
        for (int r = k + 1 + threadIdx.x; r < n; r += CWG3) y[r] -= Lf[(long long)r * n + k] * yk;
        __syncthreads();
    }
    for (int k = n - 1; k >= 0; --k) {
        const double yk = y[k] / Lf[(long long)k * n + k];
        __syncthreads();
        if (threadIdx.x == 0) y[k] = yk;
        for (int r = threadIdx.x; r < k; r += CWG3) y[r] -= Lf[(long long)k * n + r] * yk;
        __syncthreads();
    }
    for (int r = threadIdx.x; r < n; r += CWG3) a.lv[0].x[a.cidx[r]] = y[r];
    __syncthreads();
}

// levels 0..top: down (relax, residual, restrict), the coarse solve, up
// (interpolate, relax).  The caller has set b and x of level top.  On the
// small levels only a wave or two per SIMD has work, so nothing hides memory
// latency: two waves per SIMD leave the registers to issue all 54 loads of a
// 27-point row before the first use (at the default occupancy target the
// compiler keeps two in flight, and a row costs 27 trips to L2).
__global__ __launch_bounds__(CWG3) __attribute__((amdgpu_waves_per_eu(2, 2))) void k3_collapse(CArgs a)
{
    extern __shared__ double y[];
    // levels as values (not references into the argument block), so that
    // their fields stay in scalar registers across the phase loops
    for (int l = a.top; l >= 1; --l) {
        const CLev F = a.lv[l], C = a.lv[l - 1];
        wg_relax(F, a.nu1);
        wg_residual(F);
        wg_restrict(F, C);
    }
    wg_coarse(a, y);
    for (int l = 1; l <= a.top; ++l) {
        const CLev F = a.lv[l], C = a.lv[l - 1];
        wg_interp(F, C, a.rescorr);
        wg_relax(F, a.nu2);
    }
}

// ---------------------------------------------------------------------------
// The collapse of levels whose octants hold at most 64 interior vertices (9^3
// and smaller) above a coarsest level of at most SMALL_NC unknowns: the usual
// case.  Wave o holds octant o, a vertex per lane, with its whole row of the
// operator and its interpolation weights in registers, loaded once for the
// launch; the iterates and residuals live in LDS.  Such a launch is nothing but
// dependent phases, so what a phase waits for is kept out of it: the off-plane
// sums of four colours are formed together before their first, no phase reads
// memory, and none computes an index: setup packs rows, weights and indices lane
// by lane (k3_small_pack), so the launch starts with one round of coalesced
// loads.  Same terms and order as above, so the same bits; at 257^3 (levels 9^3,
// 5^3, 3^3) the launch took 153 us vertex by vertex, 24 with its indices (and
// 6 us before the first phase) in the launch, 20.6 now.
// ---------------------------------------------------------------------------
constexpr int SMALL_NC = 48, SMALL_MAXTOP = 2;

struct SRow {
    double oc[18], k[8], d, y, b, w[8], off, r;   // y: 1 / d
    int at, f;                                    // its place in LDS, the coarse corner's
    bool in;
};

// a packed level: PACK_D doubles per thread (field by field), the restriction's
// weights (27 x 64); PACK_I integers per thread: place in LDS (-1: no vertex),
// coarse corner's place, and, of the level's interior vertices in order, place in
// LDS and in the field (-1: fewer); then by coarse vertex (64) the restriction's
// fine place and its own (-1: fewer)
constexpr int PACK_D = 36, PACK_I = 4;
constexpr int PACK_DBL = PACK_D * CWG3 + 27 * 64, PACK_INT = PACK_I * CWG3 + 2 * 64;

struct SmallPack {
    const double *d[SMALL_MAXTOP + 1];
    const int *i[SMALL_MAXTOP + 1];
};

__device__ __forceinline__ int small_count(int n, int odd) { return odd ? (n - 1) / 2 : (n - 3) / 2; }

// vertex `lane` of octant o of a level (odd sides): its row and weights, all
// loads in flight
__device__ __forceinline__ void small_load(const CLev &L, const Oct &cg, int o, int lane, SRow &R)
{
    const Oct &g = L.g;
    const int na = small_count(g.nx, o & 1), nb = small_count(g.ny, (o >> 1) & 1), nc = small_count(g.nz, o >> 2);
    R.in = lane < na * nb * nc;
    const int p = R.in ? lane : 0;
    const int a = na > 0 ? p % na : 0, q = na > 0 ? p / na : 0, b = nb > 0 ? q % nb : 0, c = nb > 0 ? q / nb : 0;
    const int i = 2 * a + ((o & 1) ? 1 : 2), j = 2 * b + (((o >> 1) & 1) ? 1 : 2), k = 2 * c + ((o >> 2) ? 1 : 2);
    R.at = (k * g.ny + j) * g.nx + i;
    R.f = ((k >> 1) * cg.ny + (j >> 1)) * cg.nx + (i >> 1);
    if (!R.in) return;
    const int F = (int)g.field;
    const int t = (k >> 1) * (int)g.plane + (j >> 1) * g.px + (i >> 1), v = o * (int)g.oct + t;
#pragma unroll
    for (int s = 0; s < 9; ++s) {
        R.oc[2 * s] = L.st[(1 + s) * F + v];
        R.oc[2 * s + 1] = L.st[(1 + s) * F + nbr_rt(g, o, t, 1 - s % 3, 1 - s / 3, 1)];
    }
#pragma unroll
    for (int s = 9; s < 13; ++s) {
        R.k[2 * (s - 9)] = L.st[(1 + s) * F + v];
        R.k[2 * (s - 9) + 1] = L.st[(1 + s) * F + nbr_rt(g, o, t, 1 - s % 3, 1 - (s / 3) % 3, 0)];
    }
    R.d = L.st[v];
    R.y = 1.0 / R.d;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        R.w[m] = 1.0;
        if (!(m & ~o) && o != 0) R.w[m] = L.w[(wbase(o) + wrank(o, m)) * (int)g.oct + t];
    }
}

__device__ __forceinline__ void small_off(const SRow &R, const double *x, int nx, int nxy, double &off)
{
    off = 0.0;
#pragma unroll
    for (int s = 0; s < 9; ++s) {
        const int dx = s % 3 - 1, dy = s / 3 - 1;
        off += R.oc[2 * s] * x[R.at + dx + dy * nx - nxy];
        off += R.oc[2 * s + 1] * x[R.at - dx - dy * nx + nxy];
    }
}

__device__ __forceinline__ double small_resid(const SRow &R, const double *x, int nx)
{
    double s = R.b - R.d * x[R.at];
    s += R.off;
#pragma unroll
    for (int q = 9; q < 13; ++q) {
        const int dx = q % 3 - 1, dy = (q / 3) % 3 - 1;
        s += R.k[2 * (q - 9)] * x[R.at + dx + dy * nx];
        s += R.k[2 * (q - 9) + 1] * x[R.at - dx - dy * nx];
    }
    return s;
}

__device__ __forceinline__ void small_relax(SRow &R, double *x, int nx, int nxy, int o, int sweeps)
{
    for (int it = 0; it < sweeps; ++it)
#pragma unroll
        for (int pz = 0; pz < 2; ++pz) {
            if ((o >> 2) == pz && R.in) small_off(R, x, nx, nxy, R.off);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (o == 4 * pz + q && R.in) x[R.at] += div_by(small_resid(R, x, nx), R.d, R.y);
                __syncthreads();
            }
        }
}

// the weights of fine level F towards its coarse vertex t, slot by slot in the
// order of the restriction's sum
__device__ __forceinline__ void small_weights(const CLev &F, const Oct &c, double *wr)
{
    const Oct &g = F.g;
    const int ni = c.nx - 2, nj = c.ny - 2, n = ni * nj * (c.nz - 2);
    for (int e = threadIdx.x; e < 27 * n; e += CWG3) {
        const int s = e / n, t = e - s * n;
        const int I = 1 + t % ni, J = 1 + (t / ni) % nj, K = 1 + t / (ni * nj);
        const int ex = s % 3 - 1, ey = (s / 3) % 3 - 1, ez = s / 9 - 1;
        const int mI = (ex == -1 ? 1 : 0) | (ey == -1 ? 2 : 0) | (ez == -1 ? 4 : 0);
        wr[s * 64 + t] = weight_on(g, F.w, 2 * I + ex, 2 * J + ey, 2 * K + ez, mI);
    }
}

// pack level L (c: the level below; L.w null: the coarsest) into d and ii
__global__ __launch_bounds__(CWG3) __attribute__((amdgpu_waves_per_eu(2, 2))) void k3_small_pack(CLev L, Oct c,
                                                                                                 double *d, int *ii)
{
    const int o = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const Oct &g = L.g;
    if (L.w) {
        SRow R;
        small_load(L, c, o, lane, R);
        int q = 0;
        auto put = [&](double v) { d[q++ * CWG3 + threadIdx.x] = R.in ? v : 0.0; };
#pragma unroll
        for (int s = 0; s < 18; ++s) put(R.oc[s]);
#pragma unroll
        for (int s = 0; s < 8; ++s) put(R.k[s]);
        put(R.d);
        put(R.y);
#pragma unroll
        for (int m = 0; m < 8; ++m) put(R.w[m]);
        small_weights(L, c, d + PACK_D * CWG3);
        ii[threadIdx.x] = R.in ? R.at : -1;
        ii[CWG3 + threadIdx.x] = R.in ? R.f : 0;
        if (threadIdx.x < 64) {
            const int ni = c.nx - 2, nj = c.ny - 2, n = ni * nj * (c.nz - 2), t = threadIdx.x;
            const int I = 1 + t % ni, J = 1 + (t / ni) % nj, K = 1 + t / (ni * nj);
            ii[PACK_I * CWG3 + t] = t < n ? (2 * K * g.ny + 2 * J) * g.nx + 2 * I : 0;
            ii[PACK_I * CWG3 + 64 + t] = t < n ? (K * c.ny + J) * c.nx + I : -1;
        }
    }
    const int ni = g.nx - 2, nj = g.ny - 2, n = ni * nj * (g.nz - 2), e = threadIdx.x;
    const int i = 1 + e % ni, j = 1 + (e / ni) % nj, k = 1 + e / (ni * nj);
    ii[2 * CWG3 + e] = e < n ? (k * g.ny + j) * g.nx + i : -1;
    ii[3 * CWG3 + e] = e < n ? (int)vid(g, i, j, k) : 0;
}

// this thread's vertex of a packed level, all loads in flight
__device__ __forceinline__ void small_unpack(const double *d, const int *ii, SRow &R)
{
    const int at = ii[threadIdx.x];
    R.f = ii[CWG3 + threadIdx.x];
    int q = 0;
    auto get = [&]() { return d[q++ * CWG3 + threadIdx.x]; };
#pragma unroll
    for (int s = 0; s < 18; ++s) R.oc[s] = get();
#pragma unroll
    for (int s = 0; s < 8; ++s) R.k[s] = get();
    R.d = get();
    R.y = get();
#pragma unroll
    for (int m = 0; m < 8; ++m) R.w[m] = get();
    R.in = at >= 0;
    R.at = R.in ? at : 0;
}

// b_c = P^T r: coarse vertices on the first wave's lanes (f: the fine place of
// this lane's, to: its own, -1 without one)
__device__ __forceinline__ void small_restrict(const Oct &g, const double *r, const double *wr, double *bc, int f, int to)
{
    if (threadIdx.x < 64 && to >= 0) {
        const int nx = g.nx, nxy = g.nx * g.ny;
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < 27; ++e)
            s += wr[e * 64 + threadIdx.x] * r[f + e % 3 - 1 + ((e / 3) % 3 - 1) * nx + (e / 9 - 1) * nxy];
        bc[to] = s;
    }
    __syncthreads();
}

__device__ __forceinline__ void small_interp(const Oct &c, const SRow &R, double *x, const double *xc, int o, int rescorr)
{
    if (R.in) {
        double s = 0.0;
#pragma unroll
        for (int m = 0; m < 8; ++m)
            if (!(m & ~o)) s += R.w[m] * xc[R.f + (m & 1) + ((m >> 1) & 1) * c.nx + (m >> 2) * c.nx * c.ny];
        double xv = x[R.at] + s;
        if (o != 0 && rescorr) xv += div_by(R.r, R.d, R.y);
        x[R.at] = xv;
    }
    __syncthreads();
}

// the Cholesky substitutions of at most 64 unknowns on one wave, an unknown per
// lane (at: its place, -1 without one)
__device__ __forceinline__ void small_coarse(const double *Lf, int n, const double *b, double *x, int at)
{
    if (threadIdx.x < 64) {
        const int r = threadIdx.x;
        double y = at >= 0 ? b[at] : 0.0;
        for (int k = 0; k < n; ++k) {
            const double yk = __shfl(y, k, 64) / Lf[k * n + k];
            if (r > k && r < n) y -= Lf[r * n + k] * yk;
            if (r == k) y = yk;
        }
        for (int k = n - 1; k >= 0; --k) {
            const double yk = __shfl(y, k, 64) / Lf[k * n + k];
            if (r < k) y -= Lf[k * n + r] * yk;
            if (r == k) y = yk;
        }
        if (at >= 0) x[at] = y;
    }
    __syncthreads();
}

struct SmallLds {
    int x[SMALL_MAXTOP + 1], r[SMALL_MAXTOP + 1], b[SMALL_MAXTOP + 1], w[SMALL_MAXTOP + 1], chol, total;
};

template <int TOP>
__global__ __launch_bounds__(CWG3) __attribute__((amdgpu_waves_per_eu(2, 2))) void k3_collapse_small(CArgs a, SmallPack pk,
                                                                                                     SmallLds s)
{
    extern __shared__ double sm[];
    constexpr int NR = TOP > 0 ? TOP : 1;
    const int o = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    SRow R[NR];
    int rf[NR], rto[NR];
    double wr[NR][4];
    // every load of the launch
    const int tq = pk.i[TOP][2 * CWG3 + threadIdx.x], tv = pk.i[TOP][3 * CWG3 + threadIdx.x];
#pragma unroll
    for (int l = TOP; l >= 1; --l) {
        rf[l - 1] = pk.i[l][PACK_I * CWG3 + lane];
        rto[l - 1] = pk.i[l][PACK_I * CWG3 + 64 + lane];
        small_unpack(pk.d[l], pk.i[l], R[l - 1]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = threadIdx.x + q * CWG3;
            wr[l - 1][q] = e < 27 * 64 ? pk.d[l][PACK_D * CWG3 + e] : 0.0;
        }
    }
    const int cat = lane < a.nc ? pk.i[0][2 * CWG3 + lane] : -1;
    const CLev &T = a.lv[TOP];
    const double tx = T.x[tv], tb = T.b[tv];
    for (int e = threadIdx.x; e < s.w[0]; e += CWG3) sm[e] = 0.0;   // iterates, residuals, right-hand sides
    for (int e = threadIdx.x; e < a.nc * a.nc; e += CWG3) sm[s.chol + e] = a.chol[e];
    __syncthreads();
    if (tq >= 0) {   // the top level's right-hand side and iterate
        sm[s.x[TOP] + tq] = tx;
        sm[s.b[TOP] + tq] = tb;
    }
#pragma unroll
    for (int l = TOP; l >= 1; --l)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = threadIdx.x + q * CWG3;
            if (e < 27 * 64) sm[s.w[l] + e] = wr[l - 1][q];
        }
    __syncthreads();
#pragma unroll
    for (int l = TOP; l >= 1; --l) {
        const Oct &g = a.lv[l].g;
        SRow &Q = R[l - 1];
        double *x = sm + s.x[l];
        const int nxy = g.nx * g.ny;
        Q.b = Q.in ? sm[s.b[l] + Q.at] : 0.0;
        small_relax(Q, x, g.nx, nxy, o, a.nu1);
        if (Q.in) {
            small_off(Q, x, g.nx, nxy, Q.off);
            Q.r = small_resid(Q, x, g.nx);
            sm[s.r[l] + Q.at] = Q.r;
        }
        __syncthreads();
        small_restrict(g, sm + s.r[l], sm + s.w[l], sm + s.b[l - 1], rf[l - 1], rto[l - 1]);
    }
    small_coarse(sm + s.chol, a.nc, sm + s.b[0], sm + s.x[0], cat);
#pragma unroll
    for (int l = 1; l <= TOP; ++l) {
        const Oct &g = a.lv[l].g;
        SRow &Q = R[l - 1];
        double *x = sm + s.x[l];
        small_interp(a.lv[l - 1].g, Q, x, sm + s.x[l - 1], o, a.rescorr);
        small_relax(Q, x, g.nx, g.nx * g.ny, o, a.nu2);
    }
    if (tq >= 0) T.x[tv] = sm[s.x[TOP] + tq];
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
hipbmg_status fail3(hipbmg_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    hbmg::set_last_error(buf);
    return st;
}

#define HIP3(call)                                                                                  \
    do {                                                                                            \
        hipError_t e_ = (call);                                                                     \
        if (e_ != hipSuccess) return fail3(HIPBMG_EHIP, "%s failed: %s", #call, hipGetErrorString(e_)); \
    } while (0)

#define ST3(call)                                                                                   \
    do {                                                                                            \
        hipbmg_status s_ = (call);                                                                  \
        if (s_ != HIPBMG_OK) return s_;                                                             \
    } while (0)

inline unsigned nblk(long long n) { return (unsigned)((n + 255) / 256); }

struct Lev3 {
    Oct g;
    int npt = 27;
    int zc = 0;             // 7-point: the diagonal is formed from the connections
    double *st = nullptr;   // npt == 7: 4 fields; 27: 14 fields
    double *w = nullptr;    // NWSLOT octant slots: weights onto the next coarser level
    // the iterate's two buffers: a half sweep reads the planes it relaxes from
    // one and writes them to the other (tiles of a plane read each other's old
    // rows); x[0] holds the iterate at the start of a visit of the level
    double *x[2] = {nullptr, nullptr}, *b = nullptr, *r = nullptr;
};

constexpr int NPROF3 = 5;

}  // namespace

struct hipbmg3d_hier {
    int L = 0;
    int lstar = 0;                      // levels 0..lstar run in one workgroup
    double model_us[HIPBMG_MAX_LEVELS] = {0};
    Lev3 lv[HIPBMG_MAX_LEVELS];
    hipbmg_params prm;
    double scale = 1.0;                // the stored operator is the caller's times this power of two
    int nc = 0;
    double *d_chol = nullptr;
    long long *d_cidx = nullptr;
    SmallPack pack{};                  // the levels k3_collapse_small may run (null: not packed)
    double *d_part = nullptr;
    long long npart = 0;
    double *d_sum = nullptr;
    double *slot = nullptr, *slot_dev = nullptr;   // host-mapped {sum, tag}
    hbmg::Tags tags;
    double *d_nat = nullptr;   // plain-layout staging of the op_* entry points
    std::vector<void *> allocs;
    int cur = 0;                       // the finest iterate's buffer
    // one V-cycle and the residual norm, captured, per buffer it starts from
    hipGraph_t graph[2] = {nullptr, nullptr};
    hipGraphExec_t exec[2] = {nullptr, nullptr};
    hipStream_t cap = nullptr;         // the stream the graph is captured on (the caller's may be the null stream)
    int prof = 0;
    std::vector<hipEvent_t> evpool;
    struct ProfMark {
        int k;
        double bytes, launches;
        hipEvent_t e0, e1;
    };
    std::vector<ProfMark> marks;
    double prof_ms[NPROF3] = {0};
    double prof_n[NPROF3] = {0};
    double prof_b[NPROF3] = {0};   // algorithmic bytes of the launches timed
};

namespace {

hipbmg_status dalloc3(hipbmg3d_hier *h, double **p, long long n)
{
    void *q = nullptr;
    if (hbmg::dev_malloc(&q, (size_t)n * sizeof(double)) != hipSuccess) {
        (void)hipGetLastError();
        return fail3(HIPBMG_ENOMEM, "device allocation of %lld doubles failed", n);
    }
    h->allocs.push_back(q);
    *p = (double *)q;
    HIP3(hipMemset(q, 0, (size_t)n * sizeof(double)));
    return HIPBMG_OK;
}

void free3(hipbmg3d_hier *h)
{
    hbmg::dev_free_all(h->allocs);
    if (h->slot) {
        (void)hipDeviceSynchronize();
        hbmg::pinned_small_free(h->slot);
    }
    for (hipEvent_t e : h->evpool) (void)hipEventDestroy(e);
    for (int k = 0; k < 2; ++k) {
        if (h->exec[k]) (void)hipGraphExecDestroy(h->exec[k]);
        if (h->graph[k]) (void)hipGraphDestroy(h->graph[k]);
    }
    if (h->cap) (void)hipStreamDestroy(h->cap);
    delete h;
}

// kernel-class timing: an event pair around launches of class k, which
// move `bytes` algorithmic bytes and count as `launches` launches of the class
// (a half sweep as two of a sweep's four colour groups, the norm of the even
// planes as half a residual)
struct Mark {
    hipbmg3d_hier *h;
    int k;
    hipStream_t s;
    hipEvent_t e1 = nullptr;
    Mark(hipbmg3d_hier *h_, int k_, hipStream_t s_, double bytes = 0.0, double launches = 1.0) : h(h_), k(k_), s(s_)
    {
        if (!h->prof) return;
        const size_t need = 2 * (h->marks.size() + 1);
        while (h->evpool.size() < need) {
            hipEvent_t e;
            if (hipEventCreate(&e) != hipSuccess) {
                (void)hipGetLastError();
                h->prof = 0;
                return;
            }
            h->evpool.push_back(e);
        }
        hipEvent_t e0 = h->evpool[2 * h->marks.size()];
        e1 = h->evpool[2 * h->marks.size() + 1];
        (void)hipEventRecord(e0, s);
        h->marks.push_back({k, bytes, launches, e0, e1});
    }
    ~Mark()
    {
        if (e1) (void)hipEventRecord(e1, s);
    }
};

hipbmg_status prof_collect(hipbmg3d_hier *h)
{
    for (auto &m : h->marks) {
        float ms = 0.f;
        HIP3(hipEventSynchronize(m.e1));
        HIP3(hipEventElapsedTime(&ms, m.e0, m.e1));
        h->prof_ms[m.k] += ms;
        h->prof_n[m.k] += m.launches;
        h->prof_b[m.k] += m.bytes;
    }
    h->marks.clear();
    return HIPBMG_OK;
}

// algorithmic bytes per vertex of level f's whole grid (FP64): one
// relaxation sweep or residual reads x, b and the stencil's planes (7-point:
// C, W, S, B, or W, S, B with the diagonal formed; 27-point: 14) and writes
// x or r (the norm-only residual writes nothing)
double sweep_bytes_per_vertex(const Lev3 &f)
{
    const double planes = f.npt == 7 ? (f.zc ? 3.0 : 4.0) : 14.0;
    return 8.0 * (3.0 + planes);
}

double grid_vertices(const Lev3 &f) { return (double)f.g.nx * f.g.ny * f.g.nz; }

LArgs largs(const Lev3 &f, const Lev3 *c, int cur, int ccur)
{
    LArgs a{};
    a.g = f.g;
    a.st = f.st;
    a.b = f.b;
    a.x = f.x[cur];
    a.r = f.r;
    a.w = f.w;
    if (c) {
        a.c = c->g;
        a.xc = c->x[ccur];
        a.bc = c->b;
    }
    return a;
}

// The tiles of a level's planes of parity pz, hx halo cells to the left and hy
// halo rows below (two cells to the right and a row above always).  Whole rows
// up to PLANE_COLS cells, even shares of them beyond; as many rows as the
// workgroup holds, halved (down to two) while the launch has fewer than
// PLANE_TILES workgroups.  The large levels are bound by the bytes the tiles
// load, halo included, so their tiles are near square: 257^3 (7-point, rows of
// 128 cells) takes 89.0 ms a solve with thirds of a row by 10 rows, 91.1 with
// halves by 7; 129^3 (27-point, whole rows of 64 by 3) loses 2-6% with halves
// or smaller workgroups.  The small ones are bound by latency: 129 x 97 x 65
// takes 8.90 ms with the line at 128 or 256 workgroups, 8.97 at 512, 9.15 at
// 1024, and 3% more with tiles of one row.
constexpr int PLANE_COLS7 = 48, PLANE_COLS27 = 64, PLANE_TILES = 256;

Tile make_tile(const Oct &g, int npt, int pz, int hx, int hy)
{
    Tile t{};
    t.ncol = (g.nx - 2) / 2 + 1;
    t.nrow = (g.ny - 2) / 2 + 1;
    t.nk = pz ? (g.nz - 1) / 2 : (g.nz - 2) / 2;
    t.kk0 = pz ? 0 : 1;
    t.hx = hx;
    t.hy = hy;
    const int cols = npt == 7 ? PLANE_COLS7 : PLANE_COLS27;
    t.ntx = (t.ncol + cols - 1) / cols;
    t.tc = (t.ncol + t.ntx - 1) / t.ntx;
    t.ntx = (t.ncol + t.tc - 1) / t.tc;
    t.cw = std::min(t.ncol, t.tc + hx + 2);
    // points of a thread: two of a row (7-point), one
    const int groups = npt == 7 ? 1 : 2;
    auto shape = [&](int tr) {
        t.tr = tr;
        t.nty = (t.nrow + tr - 1) / tr;
        t.ntiles = (unsigned)((long long)t.ntx * t.nty * t.nk);
        t.rw = std::min(t.nrow, tr + hy + 1);
        t.n01 = (t.cw * t.rw + 63) / 64 * 64;
        t.n23 = (t.cw * std::min(t.nrow, tr + hy) + 63) / 64 * 64;
        return groups * (t.n01 + t.n23);
    };
    int tr = t.nrow;
    while (tr > 1 && shape(tr) > PLANE_THREADS) --tr;
    shape(tr);
    while (t.ntiles < (unsigned)PLANE_TILES && tr > 2) {
        tr = (tr + 1) / 2;
        shape(tr);
    }
    return t;
}

int tile_threads(const Tile &t, int npt) { return (npt == 7 ? 1 : 2) * (t.n01 + t.n23); }

// LDS of a tile's workgroup: the window of four octants, a cell and a row more
// than is relaxed on each side
size_t tile_lds(const Tile &t) { return 4 * (size_t)(t.cw + 2) * (t.rw + 2) * sizeof(double); }

// the norm's tiles are the last half sweep's
Tile norm_tile(const Lev3 &f, int pz) { return make_tile(f.g, f.npt, pz, pz ? 2 : 1, pz ? 1 : 0); }
long long norm_partials(const Lev3 &f)
{
    return (long long)round8(norm_tile(f, 0).ntiles) + round8(norm_tile(f, 1).ntiles);
}

template <int NPT, typename K>
hipError_t launch_tiles(K kernel, const PArgs &a, hipStream_t s)
{
    if (a.t.ntiles == 0) return hipSuccess;
    hipLaunchKernelGGL(kernel, dim3(round8(a.t.ntiles)), dim3(tile_threads(a.t, NPT)), tile_lds(a.t), s, a);
    return hipGetLastError();
}

PArgs pargs(const Lev3 &f)
{
    PArgs a{};
    a.g = f.g;
    a.st = f.st;
    a.b = f.b;
    a.r = f.r;
    a.w = f.w;
    return a;
}

template <int NPT, bool ZC>
hipError_t launch_half(int pz, bool zero, int res, const PArgs &a, hipStream_t s)
{
    if (pz == 0) {
        if (zero) return launch_tiles<NPT>(k3_plane<NPT, 0, ZC, true, 0>, a, s);
        if (res == 3) return launch_tiles<NPT>(k3_plane<NPT, 0, ZC, false, 3>, a, s);
        return launch_tiles<NPT>(k3_plane<NPT, 0, ZC, false, 0>, a, s);
    }
    if (zero)
        return res == 1 ? launch_tiles<NPT>(k3_plane<NPT, 1, ZC, true, 1>, a, s)
                        : launch_tiles<NPT>(k3_plane<NPT, 1, ZC, true, 0>, a, s);
    if (res == 1) return launch_tiles<NPT>(k3_plane<NPT, 1, ZC, false, 1>, a, s);
    if (res == 2) return launch_tiles<NPT>(k3_plane<NPT, 1, ZC, false, 2>, a, s);
    return launch_tiles<NPT>(k3_plane<NPT, 1, ZC, false, 0>, a, s);
}

// half of a relaxation of level l, the planes of parity pz from x[cur] to
// x[1 - cur]; zero: x[cur] counts as zero; res as in k3_plane (2 and 3: block
// sums into d_part)
hipbmg_status half_sweep(hipbmg3d_hier *h, int l, int cur, int pz, bool zero, int res, hipStream_t s)
{
    const Lev3 &f = h->lv[l];
    PArgs a = pargs(f);
    a.xs = f.x[cur];
    a.xo = pz ? f.x[1 - cur] : f.x[cur];
    a.xd = f.x[1 - cur];
    a.partials = h->d_part + (res == 3 ? round8(norm_tile(f, 1).ntiles) : 0);
    const bool end = res == 1 || res == 2;
    a.t = make_tile(f.g, f.npt, pz, end ? 2 : 1, end ? 1 : 0);
    // half of the sweep's vertices: two of its four colour groups {0},
    // {1,2,4}, {3,5,6}, {7}
    Mark mk(h, l == h->L - 1 ? 0 : 4, s, sweep_bytes_per_vertex(f) * grid_vertices(f) * 0.5, 2.0);
    if (f.npt == 7 && f.zc) HIP3((launch_half<7, true>(pz, zero, res, a, s)));
    else if (f.npt == 7) HIP3((launch_half<7, false>(pz, zero, res, a, s)));
    else HIP3((launch_half<27, false>(pz, zero, res, a, s)));
    return HIPBMG_OK;
}

// whether a coarse level's sweeps are one launch each (k3_sweep)
bool whole_sweeps(const hipbmg3d_hier *h, int l)
{
    const Lev3 &f = h->lv[l];
    return l < h->L - 1 && f.npt == 27 && (f.g.nz & 1) &&
           (long long)((f.g.nx - 2) / 2 + 1) * ((f.g.ny - 2) / 2 + 1) <= 64;
}

// a sweep of level l from x[cur] (zero: it counts as zero) to x[1 - cur]; resid:
// the odd planes' residual as well
hipbmg_status sweep(hipbmg3d_hier *h, int l, int cur, bool zero, bool resid, hipStream_t s)
{
    if (!whole_sweeps(h, l)) {
        ST3(half_sweep(h, l, cur, 0, zero, 0, s));
        return half_sweep(h, l, cur, 1, zero, resid ? 1 : 0, s);
    }
    const Lev3 &f = h->lv[l];
    PArgs a = pargs(f);
    a.xs = a.xo = f.x[cur];
    a.xd = f.x[1 - cur];
    Mark mk(h, 4, s);
    const dim3 grid((unsigned)((f.g.nz - 1) / 2)), block(768);
    const size_t lds = 12 * (size_t)f.g.mx * f.g.my * sizeof(double);
    if (zero && resid) hipLaunchKernelGGL((k3_sweep<true, 1>), grid, block, lds, s, a);
    else if (zero) hipLaunchKernelGGL((k3_sweep<true, 0>), grid, block, lds, s, a);
    else if (resid) hipLaunchKernelGGL((k3_sweep<false, 1>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((k3_sweep<false, 0>), grid, block, lds, s, a);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

hipbmg_status relax(hipbmg3d_hier *h, int l, int *cur, int sweeps, hipStream_t s)
{
    for (int it = 0; it < sweeps; ++it) {
        ST3(sweep(h, l, *cur, false, false, s));
        *cur = 1 - *cur;
    }
    return HIPBMG_OK;
}

// The sum of n partials into the slot, tagged `tag` (0: the last tag plus 1).
// Up to 2048 in one launch, more in two stages of fixed shape (deterministic).
hipbmg_status reduce_sum(hipbmg3d_hier *h, const double *partials, long long n, double tag, hipStream_t s)
{
    const long long nb = std::min<long long>(256, (n + 2047) / 2048);
    if (nb > 1) {
        const long long chunk = (n + nb - 1) / nb;
        hipLaunchKernelGGL(k3_reduce, dim3((unsigned)nb), dim3(256), 0, s, partials, n, chunk, h->d_sum + 8);
        partials = h->d_sum + 8;
        n = nb;
    }
    hipLaunchKernelGGL(k3_sum_out, dim3(1), dim3(256), 0, s, partials, n, h->d_sum, tag, h->slot_dev);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

// wait for the sum tagged `tag`
hipbmg_status wait_sum(hipbmg3d_hier *h, double tag, hipStream_t s, double *out)
{
    const hipError_t e = hbmg::wait_tag(h->slot + 1, tag, s);
    if (e != hipSuccess) return fail3(HIPBMG_EHIP, "a norm did not arrive: %s", hipGetErrorString(e));
    *out = h->slot[0];
    return HIPBMG_OK;
}

// residual r = b - A x[cur] of level l
hipbmg_status residual(hipbmg3d_hier *h, int l, int cur, hipStream_t s)
{
    const Lev3 &f = h->lv[l];
    const LArgs a = largs(f, nullptr, cur, 0);
    const dim3 grid(8 * nblk(f.g.oct)), block(256);   // a multiple of 8, octants interleaved
    Mark mk(h, 4, s);
    if (f.npt == 7) hipLaunchKernelGGL((k3_resid<7>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k3_resid<27>), grid, block, 0, s, a);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

// ||b - A x[cur]||^2 of the finest level into the slot.  The block sums of the
// planes of a parity that a half sweep has left in d_part already (have_odd,
// have_even) are the same bits this forms.
hipbmg_status norm(hipbmg3d_hier *h, int cur, bool have_odd, bool have_even, hipStream_t s)
{
    const Lev3 &f = h->lv[h->L - 1];
    PArgs a = pargs(f);
    a.xs = a.xo = f.x[cur];
    for (int pz = 0; pz < 2; ++pz) {
        if (pz ? have_odd : have_even) continue;
        a.t = norm_tile(f, pz);
        a.partials = h->d_part + (pz ? 0 : round8(norm_tile(f, 1).ntiles));
        Mark mk(h, 1, s, (sweep_bytes_per_vertex(f) - 8.0) * grid_vertices(f) * 0.5, 0.5);
        if (f.npt == 7 && f.zc)
            HIP3(pz ? launch_tiles<7>(k3_plane_resid<7, 1, true, true>, a, s)
                    : launch_tiles<7>(k3_plane_resid<7, 0, true, true>, a, s));
        else if (f.npt == 7)
            HIP3(pz ? launch_tiles<7>(k3_plane_resid<7, 1, false, true>, a, s)
                    : launch_tiles<7>(k3_plane_resid<7, 0, false, true>, a, s));
        else
            HIP3(pz ? launch_tiles<27>(k3_plane_resid<27, 1, false, true>, a, s)
                    : launch_tiles<27>(k3_plane_resid<27, 0, false, true>, a, s));
    }
    return reduce_sum(h, h->d_part, norm_partials(f), 0.0, s);
}

// b_{l-1} = P^T r_l, and x_{l-1} = 0 if zero
hipbmg_status restrict_to(hipbmg3d_hier *h, int l, bool zero, hipStream_t s)
{
    LArgs a = largs(h->lv[l], &h->lv[l - 1], 0, 0);
    if (zero) a.xcz = h->lv[l - 1].x[0];
    // reads r and the 26 weights per coarse cell (3.25 per fine vertex),
    // writes the coarse right-hand side and the zero coarse iterate
    Mark mk(h, l == h->L - 1 ? 2 : 4, s, 8.0 * (1.0 + 3.25 + 0.25) * grid_vertices(h->lv[l]));
    hipLaunchKernelGGL(k3_restrict, dim3(8 * nblk(a.c.oct)), dim3(256), 0, s, a);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

// the same, with the even planes' residual of x[cur] formed on the way (the
// odd planes' is in r)
hipbmg_status residual_restrict(hipbmg3d_hier *h, int l, int cur, bool zero, hipStream_t s)
{
    const Lev3 &f = h->lv[l], &c = h->lv[l - 1];
    PArgs a = pargs(f);
    a.xs = a.xo = f.x[cur];
    a.c = c.g;
    a.bc = c.b;
    a.xcz = zero ? c.x[0] : nullptr;
    a.t = make_tile(f.g, f.npt, 0, 1, 1);
    Mark mk(h, l == h->L - 1 ? 2 : 4, s,
            (0.5 * sweep_bytes_per_vertex(f) + 8.0 * (0.5 + 3.25 + 0.125)) * grid_vertices(f));
    if (f.npt == 7 && f.zc) HIP3((launch_tiles<7>(k3_plane_resid<7, 0, true, false>, a, s)));
    else if (f.npt == 7) HIP3((launch_tiles<7>(k3_plane_resid<7, 0, false, false>, a, s)));
    else HIP3((launch_tiles<27>(k3_plane_resid<27, 0, false, false>, a, s)));
    return HIPBMG_OK;
}

// x[cur] += P x_{l-1}[ccur] (+ r/C)
hipbmg_status interp_from(hipbmg3d_hier *h, int l, int cur, int ccur, int rescorr, hipStream_t s)
{
    const Lev3 &f = h->lv[l];
    LArgs a = largs(f, &h->lv[l - 1], cur, ccur);
    a.rescorr = rescorr;
    const dim3 grid(round8(nblk(f.g.oct)), 8), block(256);
    // reads and writes x, reads r, C, the weights and the coarse iterate
    Mark mk(h, l == h->L - 1 ? 3 : 4, s, 8.0 * (2.0 + 1.0 + 1.0 + 3.25 + 0.125) * grid_vertices(f));
    if (f.npt == 7) hipLaunchKernelGGL((k3_interp<7>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k3_interp<27>), grid, block, 0, s, a);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

// whether levels 0..top take the register-resident collapse, and its LDS: every
// level above the coarsest with 27 points, odd sides and at most 64 interior
// vertices in its largest octant (the one of all odd indices), which caps top
// at 2; at most SMALL_NC unknowns on the coarsest; 64 KB of LDS
bool small_collapse(const hipbmg3d_hier *h, int top, SmallLds *s)
{
    if (top > SMALL_MAXTOP || h->nc > SMALL_NC || h->nc < 1) return false;
    for (int l = 1; l <= top; ++l) {
        const Oct &g = h->lv[l].g;
        if (h->lv[l].npt != 27 || !(g.nx & 1) || !(g.ny & 1) || !(g.nz & 1) ||
            (long long)((g.nx - 1) / 2) * ((g.ny - 1) / 2) * ((g.nz - 1) / 2) > 64)
            return false;
    }
    int at = 0;
    for (int l = 0; l <= top; ++l) {
        const Oct &g = h->lv[l].g;
        const int n = g.nx * g.ny * g.nz;
        s->x[l] = at;
        s->b[l] = at + n;
        s->r[l] = at + 2 * n;
        at += (l > 0 ? 3 : 2) * n;
    }
    s->w[0] = at;   // what starts as zero ends here
    for (int l = 1; l <= top; ++l) {
        s->w[l] = at;
        at += 27 * 64;
    }
    s->chol = at;
    s->total = at + h->nc * h->nc;
    return (size_t)s->total * sizeof(double) <= 64 * 1024;
}

// pack the levels that k3_collapse_small may run, once their operators are complete
hipbmg_status small_pack(hipbmg3d_hier *h, hipStream_t s)
{
    SmallLds sl;
    for (int l = 0; l < h->L && small_collapse(h, l, &sl); ++l) {
        const Lev3 &v = h->lv[l];
        double *d = nullptr, *i = nullptr;
        if (l > 0) ST3(dalloc3(h, &d, PACK_DBL));
        ST3(dalloc3(h, &i, (PACK_INT + 1) / 2));
        const CLev c{v.g, v.npt, v.st, l > 0 ? v.w : nullptr, v.x[0], v.b, v.r};
        hipLaunchKernelGGL(k3_small_pack, dim3(1), dim3(CWG3), 0, s, c, h->lv[l > 0 ? l - 1 : 0].g, d, (int *)i);
        HIP3(hipGetLastError());
        h->pack.d[l] = d;
        h->pack.i[l] = (const int *)i;
    }
    return HIPBMG_OK;
}

// levels 0..top in one workgroup (top = 0: the coarse solve alone)
hipbmg_status collapse(hipbmg3d_hier *h, int top, hipStream_t s)
{
    CArgs a{};
    for (int l = 0; l <= top; ++l) {
        const Lev3 &v = h->lv[l];
        a.lv[l] = CLev{v.g, v.npt, v.st, v.w, v.x[0], v.b, v.r};
    }
    a.top = top;
    a.chol = h->d_chol;
    a.cidx = h->d_cidx;
    a.nc = h->nc;
    a.nu1 = h->prm.nu1;
    a.nu2 = h->prm.nu2;
    a.rescorr = h->prm.residual_correction;
    Mark mk(h, 4, s);
    SmallLds sl;
    if (small_collapse(h, top, &sl)) {
        const dim3 one(1), wg(CWG3);
        const size_t lds = (size_t)sl.total * sizeof(double);
        if (top == 0) hipLaunchKernelGGL(k3_collapse_small<0>, one, wg, lds, s, a, h->pack, sl);
        else if (top == 1) hipLaunchKernelGGL(k3_collapse_small<1>, one, wg, lds, s, a, h->pack, sl);
        else hipLaunchKernelGGL(k3_collapse_small<2>, one, wg, lds, s, a, h->pack, sl);
        HIP3(hipGetLastError());
        return HIPBMG_OK;
    }
    hipLaunchKernelGGL(k3_collapse, dim3(1), dim3(CWG3), (size_t)std::max(h->nc, 1) * sizeof(double), s, a);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

// Algorithm 1 on level l; the iterate starts in x[0] (on the finest level in
// x[h->cur], and from zero on all others) and ends in x[*end].  begun: the
// first sweep has been done; norm_odd: the last one also leaves the odd
// planes' part of the norm in d_part.
hipbmg_status vcycle(hipbmg3d_hier *h, int l, hipStream_t s, int *end = nullptr, bool begun = false,
                     bool norm_odd = false)
{
    const bool fine = l == h->L - 1;
    int cur = fine ? h->cur : 0;
    if (end) *end = cur;
    if (l <= h->lstar) return collapse(h, l, s);
    const int nu1 = h->prm.nu1, nu2 = h->prm.nu2;
    for (int it = 0; it < nu1; ++it) {
        const bool zero = !fine && it == 0;
        if (!(begun && it == 0)) {
            ST3(sweep(h, l, cur, zero, it == nu1 - 1, s));
        }
        cur = 1 - cur;
    }
    // the coarse iterate's zeros are stored only for what reads them: the
    // collapsed workgroup, or a level without pre-relaxations
    const bool zero = l - 1 <= h->lstar || nu1 == 0;
    if (nu1 > 0) {
        ST3(residual_restrict(h, l, cur, zero, s));
    } else {
        ST3(residual(h, l, cur, s));
        ST3(restrict_to(h, l, zero, s));
    }
    int ccur = 0;
    ST3(vcycle(h, l - 1, s, &ccur));
    ST3(interp_from(h, l, cur, ccur, h->prm.residual_correction, s));
    for (int it = 0; it < nu2; ++it) {
        if (norm_odd && it == nu2 - 1) {
            ST3(half_sweep(h, l, cur, 0, false, 0, s));
            ST3(half_sweep(h, l, cur, 1, false, 2, s));
        } else {
            ST3(sweep(h, l, cur, false, false, s));
        }
        cur = 1 - cur;
    }
    if (end) *end = cur;
    return HIPBMG_OK;
}

// the finest level's cycles overlap: a cycle ends with the first sweep of the
// next one, which writes the other buffer (the iterate stays whole where a cycle
// was the last).  Its first half sums the squares of the residual it starts
// from, so the norm's even planes cost no pass of their own; the second runs
// while the host sees the norm and enqueues the next cycle.  Not where kernel
// timing is on, which times the norm as a launch of its own.
bool overlapped(const hipbmg3d_hier *h) { return h->L - 1 > h->lstar && h->prm.nu1 > 0 && !h->prof; }

hipbmg_status second_half(hipbmg3d_hier *h, int cur, hipStream_t s)
{
    return half_sweep(h, h->L - 1, cur, 1, false, h->prm.nu1 == 1 ? 1 : 0, s);
}

hipbmg_status enqueue_cycle(hipbmg3d_hier *h, hipStream_t s, int *end)
{
    const bool norm_odd = h->L - 1 > h->lstar && h->prm.nu2 > 0, over = overlapped(h);
    ST3(vcycle(h, h->L - 1, s, end, over, norm_odd));
    if (over) ST3(half_sweep(h, h->L - 1, *end, 0, false, 3, s));
    ST3(norm(h, *end, norm_odd, over, s));
    return over ? second_half(h, *end, s) : HIPBMG_OK;
}

// one cycle and the finest residual norm (into the slot); replayed from a
// captured graph (one per buffer the finest iterate starts from) unless
// use_graph is 0 or kernel timing is on
hipbmg_status cycle_and_norm(hipbmg3d_hier *h, hipStream_t s)
{
    const int k = h->cur;
    int end = k;
    if (!h->prm.use_graph || h->prof) {
        ST3(enqueue_cycle(h, s, &end));
        h->cur = end;
        return HIPBMG_OK;
    }
    if (!h->exec[k]) {
        if (!h->cap) HIP3(hipStreamCreateWithFlags(&h->cap, hipStreamNonBlocking));
        hipStream_t c = h->cap;
        HIP3(hipStreamBeginCapture(c, hipStreamCaptureModeThreadLocal));
        const hipbmg_status st = enqueue_cycle(h, c, &end);
        hipGraph_t g = nullptr;
        const hipError_t e2 = hipStreamEndCapture(c, &g);
        if (st != HIPBMG_OK || e2 != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            return st != HIPBMG_OK ? st : fail3(HIPBMG_EHIP, "graph capture failed: %s", hipGetErrorString(e2));
        }
        h->graph[k] = g;
        HIP3(hipGraphInstantiate(&h->exec[k], g, nullptr, nullptr, 0));
    }
    HIP3(hipGraphLaunch(h->exec[k], s));
    if (h->L - 1 > h->lstar) h->cur = k ^ ((h->prm.nu1 + h->prm.nu2) & 1);
    return HIPBMG_OK;
}

hipbmg_status to_oct(const Oct &g, const double *nat, double *out, int interior_only, hipStream_t s,
                     double scale = 1.0, int *tiny = nullptr)
{
    hipLaunchKernelGGL(k3_to_oct, dim3(nblk((long long)g.nx * g.ny * g.nz)), dim3(256), 0, s, nat, out, g,
                       interior_only, scale, tiny);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

hipbmg_status from_oct(const Oct &g, const double *in, double *nat, hipStream_t s, double scale = 1.0)
{
    hipLaunchKernelGGL(k3_from_oct, dim3(nblk((long long)g.nx * g.ny * g.nz)), dim3(256), 0, s, in, nat, g,
                       scale);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

// host copy of A(p, p+d) for the coarsest assembly
void host_entries(const std::vector<double> &st, int npt, const Oct &g, int i, int j, int k, double e[27])
{
    const long long v = vid(g, i, j, k), F = g.field;
    for (int o = 0; o < 27; ++o) e[o] = 0.0;
    e[13] = st[v];
    if (npt == 7) {
        e[12] = -st[F + v];
        e[14] = -st[F + vid(g, i + 1, j, k)];
        e[10] = -st[2 * F + v];
        e[16] = -st[2 * F + vid(g, i, j + 1, k)];
        e[4] = -st[3 * F + v];
        e[22] = -st[3 * F + vid(g, i, j, k + 1)];
    } else {
        for (int o = 0; o < 13; ++o) {
            const int dx = o % 3 - 1, dy = (o / 3) % 3 - 1, dz = o / 9 - 1;
            e[o] = -st[(1 + o) * F + v];
            e[26 - o] = -st[(1 + o) * F + vid(g, i - dx, j - dy, k - dz)];
        }
    }
}

constexpr int MAX_COARSE3 = 4096;

hipbmg_status factor_coarsest(hipbmg3d_hier *h, hipStream_t s)
{
    const Lev3 &c = h->lv[0];
    const Oct &g = c.g;
    const int nf = c.npt == 7 ? 4 : 14;
    std::vector<double> st((size_t)nf * g.field);
    HIP3(hipMemcpyAsync(st.data(), c.st, st.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    HIP3(hipStreamSynchronize(s));
    std::vector<long long> cidx;
    std::vector<int> num((size_t)g.nx * g.ny * g.nz, -1);
    for (int k = 1; k <= g.nz - 2; ++k)
        for (int j = 1; j <= g.ny - 2; ++j)
            for (int i = 1; i <= g.nx - 2; ++i) {
                num[((size_t)k * g.ny + j) * g.nx + i] = (int)cidx.size();
                cidx.push_back(vid(g, i, j, k));
            }
    const int n = (int)cidx.size();
    if (n > MAX_COARSE3) return fail3(HIPBMG_EINVAL, "coarsest level has %d unknowns (at most %d)", n, MAX_COARSE3);
    std::vector<double> M((size_t)n * n, 0.0);
    for (int k = 1; k <= g.nz - 2; ++k)
        for (int j = 1; j <= g.ny - 2; ++j)
            for (int i = 1; i <= g.nx - 2; ++i) {
                double e[27];
                host_entries(st, c.npt, g, i, j, k, e);
                const int row = num[((size_t)k * g.ny + j) * g.nx + i];
                for (int o = 0; o < 27; ++o) {
                    const int qi = i + o % 3 - 1, qj = j + (o / 3) % 3 - 1, qk = k + o / 9 - 1;
                    if (!inner(g, qi, qj, qk)) continue;
                    M[(size_t)row * n + num[((size_t)qk * g.ny + qj) * g.nx + qi]] = e[o];
                }
            }
    for (int k = 0; k < n; ++k) {
        double d = M[(size_t)k * n + k];
        for (int m = 0; m < k; ++m) d -= M[(size_t)k * n + m] * M[(size_t)k * n + m];
        if (!(d > 0.0)) return fail3(HIPBMG_ENOTSPD, "coarsest operator not positive definite (pivot %d)", k);
        d = std::sqrt(d);
        M[(size_t)k * n + k] = d;
        for (int r = k + 1; r < n; ++r) {
            double v = M[(size_t)r * n + k];
            for (int m = 0; m < k; ++m) v -= M[(size_t)r * n + m] * M[(size_t)k * n + m];
            M[(size_t)r * n + k] = v / d;
        }
    }
    h->nc = n;
    ST3(dalloc3(h, &h->d_chol, std::max((long long)n * n, 1LL)));
    double *ci = nullptr;
    ST3(dalloc3(h, &ci, std::max(n, 1)));
    h->d_cidx = (long long *)ci;
    if (n > 0) {
        HIP3(hipMemcpyAsync(h->d_chol, M.data(), M.size() * sizeof(double), hipMemcpyHostToDevice, s));
        HIP3(hipMemcpyAsync(h->d_cidx, cidx.data(), cidx.size() * sizeof(long long), hipMemcpyHostToDevice, s));
        HIP3(hipStreamSynchronize(s));
    }
    return HIPBMG_OK;
}

bool odd_ok(int n) { return n >= 3 && (n & 1); }

// mean time (ms) of `reps` repetitions of f on stream s, after one warm-up
template <typename Fn>
hipbmg_status time_ms(hipStream_t s, int reps, Fn f, double *ms)
{
    hipEvent_t e0, e1;
    ST3(f());
    HIP3(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return fail3(HIPBMG_EHIP, "hipEventCreate failed");
    }
    hipbmg_status st = HIPBMG_OK;
    if (hipEventRecord(e0, s) != hipSuccess) st = fail3(HIPBMG_EHIP, "hipEventRecord failed");
    for (int r = 0; r < reps && st == HIPBMG_OK; ++r) st = f();
    float t = 0.f;
    if (st == HIPBMG_OK && (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                            hipEventElapsedTime(&t, e0, e1) != hipSuccess))
        st = fail3(HIPBMG_EHIP, "event timing failed");
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    *ms = t / reps;
    return st;
}

// The model's choice of l*.  For the levels up to 9^3-ish (l <= 3) both of a
// level's terms are measured: its cost inside the workgroup as the growth of
// the collapse launch from top = l-1 to top = l, and its grid-wide cost as one
// eager visit of level l on top of the collapse of levels 0..l-1 minus that
// collapse.  Larger levels take the model's formulas.  The levels hold zeros
// while this runs, which the solve overwrites.
hipbmg_status choose_collapse(hipbmg3d_hier *h, const hbmg::ModelLevel3 *ml, int lcap, hipStream_t s)
{
    const int L = h->L;
    double t_us[HIPBMG_MAX_LEVELS];
    hbmg::model3_choose(ml, L, h->prm.nu1, h->prm.nu2, h->nc, hbmg::model_params(), lcap, t_us);
    const int m = std::min(3, lcap);
    double tc[4] = {0}, tw[4] = {0}, tg[4] = {0};
    for (int top = 0; top <= m; ++top)
        ST3(time_ms(s, 5, [&]() { return collapse(h, top, s); }, &tc[top]));
    for (int l = 1; l <= m; ++l) {
        double t = 0.0;
        h->lstar = l - 1;
        const hipbmg_status st = time_ms(s, 5, [&]() { return vcycle(h, l, s); }, &t);
        h->lstar = 0;
        ST3(st);
        tw[l] = 1e3 * (tc[l] - tc[l - 1]);
        tg[l] = 1e3 * t - 1e3 * tc[l - 1];
    }
    int best = 0;
    for (int ls = 0; ls <= lcap; ++ls) {
        const hbmg::ModelParams &mp = hbmg::model_params();
        double t = 1e3 * tc[0];
        if (ls <= m) {
            for (int l = 1; l < L; ++l) {
                if (l <= m) t += l <= ls ? tw[l] : tg[l];
                else t += hbmg::model3_grid_level_us(ml[l], h->prm.nu1, h->prm.nu2, mp);
            }
        } else {
            // the model's path with its base and its small-level terms replaced by the measured ones
            t += t_us[ls] - hbmg::model_base_us(h->nc, 8, mp);
            for (int l = 1; l <= m; ++l) t += tw[l] - hbmg::model3_wg_level_us(ml[l], h->prm.nu1, h->prm.nu2, mp);
        }
        h->model_us[ls] = t;
        if (t < h->model_us[best]) best = ls;
    }
    h->lstar = best;
    return HIPBMG_OK;
}

}  // namespace

// ---------------------------------------------------------------------------
// C interface
// ---------------------------------------------------------------------------
extern "C" hipbmg_status hipbmg3d_fv7_from_cells(int nx, int ny, int nz, const double *cell, double *planes_out,
                                                 void *stream)
{
    if (!cell || !planes_out) return fail3(HIPBMG_EINVAL, "null argument");
    if (nx < 3 || ny < 3 || nz < 3) return fail3(HIPBMG_EINVAL, "grid too small");
    hipStream_t s = (hipStream_t)stream;
    const long long n = (long long)nx * ny * nz;
    hipLaunchKernelGGL(k3_fv7, dim3(nblk(n)), dim3(256), 0, s, cell, nx, ny, nz, planes_out);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

// Build a hierarchy whose stored operator is the caller's times scale; *tiny is
// set where scale = 1 leaves reciprocals of its diagonal out of range.
static hipbmg_status build_hierarchy3(int nx, int ny, int nz, int npt, const double *planes, const hipbmg_params &prm,
                                      hipStream_t s, double scale, int *tiny, hipbmg3d_hier **out)
{
    int sx[HIPBMG_MAX_LEVELS], sy[HIPBMG_MAX_LEVELS], sz[HIPBMG_MAX_LEVELS], L = 1;
    sx[0] = nx;
    sy[0] = ny;
    sz[0] = nz;
    while (sx[L - 1] > prm.coarsest_n && sy[L - 1] > prm.coarsest_n && sz[L - 1] > prm.coarsest_n &&
           (sx[L - 1] & 1) && (sy[L - 1] & 1) && (sz[L - 1] & 1) && L < HIPBMG_MAX_LEVELS) {
        sx[L] = (sx[L - 1] + 1) / 2;
        sy[L] = (sy[L - 1] + 1) / 2;
        sz[L] = (sz[L - 1] + 1) / 2;
        ++L;
    }
    {
        const Oct g0 = make_oct(sx[L - 1], sy[L - 1], sz[L - 1]);
        const long long nc = (long long)(g0.nx - 2) * (g0.ny - 2) * (g0.nz - 2);
        if (nc > MAX_COARSE3)
            return fail3(HIPBMG_EINVAL, "coarsest level %dx%dx%d has %lld unknowns (at most %d)", g0.nx, g0.ny,
                         g0.nz, nc, MAX_COARSE3);
    }
    auto t0 = std::chrono::steady_clock::now();
    hipbmg3d_hier *h = new hipbmg3d_hier();
    h->L = L;
    h->prm = prm;
    h->scale = scale;
    auto bail = [&](hipbmg_status st) {
        free3(h);
        return st;
    };
    hipbmg_status st;
    for (int l = 0; l < L; ++l) {
        Lev3 &v = h->lv[l];
        v.g = make_oct(sx[L - 1 - l], sy[L - 1 - l], sz[L - 1 - l]);
        v.npt = (l == L - 1) ? npt : 27;
        const int nf = v.npt == 7 ? 4 : 14;
        if ((st = dalloc3(h, &v.st, nf * v.g.field)) != HIPBMG_OK) return bail(st);
        for (int k = 0; k < 2; ++k)
            if ((st = dalloc3(h, &v.x[k], v.g.field)) != HIPBMG_OK) return bail(st);
        if ((st = dalloc3(h, &v.b, v.g.field)) != HIPBMG_OK) return bail(st);
        if ((st = dalloc3(h, &v.r, v.g.field)) != HIPBMG_OK) return bail(st);
        if (l >= 1 && (st = dalloc3(h, &v.w, NWSLOT * v.g.oct)) != HIPBMG_OK) return bail(st);
    }
    const Lev3 &top = h->lv[L - 1];
    const long long nnat = (long long)nx * ny * nz;
    if ((st = dalloc3(h, &h->d_nat, nnat)) != HIPBMG_OK) return bail(st);
    h->npart = (long long)nblk(top.g.field) + norm_partials(top) + 8;
    if ((st = dalloc3(h, &h->d_part, h->npart)) != HIPBMG_OK) return bail(st);
    if ((st = dalloc3(h, &h->d_sum, 8 + 256)) != HIPBMG_OK) return bail(st);
    if (hbmg::pinned_small((void **)&h->slot, (void **)&h->slot_dev, 3 * sizeof(double)) != hipSuccess ||
        !h->slot_dev) {
        (void)hipGetLastError();
        return bail(fail3(HIPBMG_ENOMEM, "host-mapped allocation failed"));
    }
    h->slot[0] = h->slot[1] = h->slot[2] = 0.0;
    int *const d_tiny = reinterpret_cast<int *>(h->slot_dev + 2);   // read after the setup's last wait
    // the finest operator in the octant layout
    const int nf = npt == 7 ? 4 : 14;
    for (int q = 0; q < nf; ++q)
        if ((st = to_oct(top.g, planes + q * nnat, top.st + q * top.g.field, 0, s, scale, q == 0 ? d_tiny : nullptr)) !=
            HIPBMG_OK)
            return bail(st);
    // a 7-point finest operator whose diagonal is the sum of its six
    // connections (finite volumes of pure diffusion): its relaxation and
    // residual kernels form the diagonal instead of loading it
    // (HIPBMG_NO_ZEXC=1: always load)
    if (npt == 7) {
        int noz = 0;
        if (const char *e = std::getenv("HIPBMG_NO_ZEXC")) noz = std::atoi(e);
        if (!noz) {
            int ok = 0;
            double *dflag = nullptr;   // one double of device memory holds the int flag
            if ((st = dalloc3(h, &dflag, 1)) != HIPBMG_OK) return bail(st);
            int *d_flag = reinterpret_cast<int *>(dflag);
            hipLaunchKernelGGL(k3_set_int, dim3(1), dim3(1), 0, s, d_flag, 1);
            hipLaunchKernelGGL(k3_zero_excess7, dim3(8 * nblk(top.g.oct)), dim3(256), 0, s, top.g,
                               (const double *)top.st, d_flag);
            if (hipGetLastError() != hipSuccess ||
                hipMemcpyAsync(&ok, d_flag, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess)
                return bail(fail3(HIPBMG_EHIP, "zero-excess check failed"));
            h->lv[L - 1].zc = ok;
        }
    }
    // interpolation and Galerkin products, finest to coarsest
    for (int l = L - 1; l >= 1; --l) {
        Lev3 &f = h->lv[l], &c = h->lv[l - 1];
        WArgs wa{Sten{f.st, f.npt, f.g}, f.w, c.g};
        hipLaunchKernelGGL(k3_weights<1>, dim3(nblk(f.g.oct), 3), dim3(256), 0, s, wa);
        hipLaunchKernelGGL(k3_weights<2>, dim3(nblk(f.g.oct), 3), dim3(256), 0, s, wa);
        hipLaunchKernelGGL(k3_weights<3>, dim3(nblk(f.g.oct), 1), dim3(256), 0, s, wa);
        RArgs ra{Sten{f.st, f.npt, f.g}, f.w, c.g, c.st};
        hipLaunchKernelGGL(k3_rap, dim3(nblk(c.g.field)), dim3(256), 0, s, ra);
        if (hipGetLastError() != hipSuccess) return bail(fail3(HIPBMG_EHIP, "setup kernel launch failed"));
    }
    if ((st = factor_coarsest(h, s)) != HIPBMG_OK) return bail(st);
    if ((st = small_pack(h, s)) != HIPBMG_OK) return bail(st);
    // the collapse level: forced, or the model's argmin (section 3's model
    // with 3D counts).  Its terms for the small levels are measured here on
    // the hierarchy's own launches; larger levels use the process-wide
    // calibrated machine parameters.
    {
        int lcap = std::min(L - 1, MAXC3 - 1);
        // 32-bit indices in the workgroup: every plane offset of a collapsed level
        while (lcap > 0 && (long long)(h->lv[lcap].npt == 7 ? 4 : 14) * h->lv[lcap].g.field >= (1LL << 31)) --lcap;
        hbmg::ModelLevel3 ml[HIPBMG_MAX_LEVELS];
        for (int l = 0; l < L; ++l)
            ml[l] = hbmg::ModelLevel3{h->lv[l].g.nx, h->lv[l].g.ny, h->lv[l].g.nz, h->lv[l].npt};
        if (prm.collapse_level >= 0) {
            if (prm.collapse_level > lcap)
                return bail(fail3(HIPBMG_EINVAL, "collapse_level %d out of range (at most %d)", prm.collapse_level,
                                  lcap));
            hbmg::model3_choose(ml, L, prm.nu1, prm.nu2, h->nc, hbmg::model_params(), lcap, h->model_us);
            h->lstar = prm.collapse_level;
        } else if ((st = choose_collapse(h, ml, lcap, s)) != HIPBMG_OK) {
            return bail(st);
        }
    }
    if (hipStreamSynchronize(s) != hipSuccess) return bail(fail3(HIPBMG_EHIP, "setup failed on the device"));
    (void)t0;
    *tiny = *reinterpret_cast<const volatile int *>(h->slot + 2);
    *out = h;
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_setup(int nx, int ny, int nz, int npt, const double *planes,
                                        const hipbmg_params *params, void *stream, hipbmg3d_handle *out)
{
    if (!out || !planes) return fail3(HIPBMG_EINVAL, "null argument");
    *out = nullptr;
    if (!odd_ok(nx) || !odd_ok(ny) || !odd_ok(nz)) return fail3(HIPBMG_EINVAL, "sizes must be odd and >= 3");
    if (npt != 7 && npt != 27) return fail3(HIPBMG_EINVAL, "npt must be 7 or 27");
    hipbmg_params prm;
    hipbmg_default_params(&prm);
    if (params) prm = *params;
    if (prm.nu1 < 0 || prm.nu2 < 0 || prm.nu1 + prm.nu2 < 1 || prm.coarsest_n < 3 || prm.max_cycles < 1 ||
        prm.max_cycles > HIPBMG_MAX_HIST)
        return fail3(HIPBMG_EINVAL, "bad parameters");
    if (prm.precision != HIPBMG_FP64) return fail3(HIPBMG_EINVAL, "the 3D path runs in FP64 only");
    // as in 2D, an operator with diagonals so small that their reciprocals
    // overflow is built again, scaled by a power of two
    for (double scale = 1.0;; scale = hbmg::TINY_SCALE) {
        hipbmg3d_hier *h = nullptr;
        int tiny = 0;
        ST3(build_hierarchy3(nx, ny, nz, npt, planes, prm, (hipStream_t)stream, scale, &tiny, &h));
        if (!tiny || scale != 1.0) {
            *out = h;
            return HIPBMG_OK;
        }
        free3(h);
    }
}

extern "C" hipbmg_status hipbmg3d_destroy(hipbmg3d_handle h)
{
    if (h) free3(h);
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_num_levels(hipbmg3d_handle h, int *levels_host)
{
    if (!h || !levels_host) return fail3(HIPBMG_EINVAL, "null argument");
    *levels_host = h->L;
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_level_size(hipbmg3d_handle h, int l, int *nx_host, int *ny_host, int *nz_host)
{
    if (!h || !nx_host || !ny_host || !nz_host) return fail3(HIPBMG_EINVAL, "null argument");
    if (l < 0 || l >= h->L) return fail3(HIPBMG_EINVAL, "level %d out of range", l);
    *nx_host = h->lv[l].g.nx;
    *ny_host = h->lv[l].g.ny;
    *nz_host = h->lv[l].g.nz;
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_get_stencil(hipbmg3d_handle h, int l, double *out, void *stream)
{
    if (!h || !out) return fail3(HIPBMG_EINVAL, "null argument");
    if (l < 0 || l >= h->L) return fail3(HIPBMG_EINVAL, "level %d out of range", l);
    const Lev3 &v = h->lv[l];
    const long long n = (long long)v.g.nx * v.g.ny * v.g.nz;
    hipLaunchKernelGGL(k3_stencil_out, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, Sten{v.st, v.npt, v.g},
                       out, 1.0 / h->scale);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_get_interp(hipbmg3d_handle h, int l, double *out, void *stream)
{
    if (!h || !out) return fail3(HIPBMG_EINVAL, "null argument");
    if (l < 1 || l >= h->L) return fail3(HIPBMG_EINVAL, "level %d has no interpolation", l);
    const Lev3 &v = h->lv[l];
    const long long n = (long long)v.g.nx * v.g.ny * v.g.nz;
    hipLaunchKernelGGL(k3_interp_out, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, v.g,
                       (const double *)v.w, out);
    HIP3(hipGetLastError());
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_solve(hipbmg3d_handle h, const double *b, double *u, double tol, void *stream,
                                        hipbmg_info *info)
{
    if (!h || !b || !u) return fail3(HIPBMG_EINVAL, "null argument");
    if (!(tol >= 0.0)) return fail3(HIPBMG_EINVAL, "bad tolerance");
    hipStream_t s = (hipStream_t)stream;
    auto t0 = std::chrono::steady_clock::now();
    Lev3 &f = h->lv[h->L - 1];
    hbmg::Drain drain{s};
    // the first sweep waits for ||b||, which comes while u is on its way in: a
    // solve of b = 0 does not pay for it
    ST3(to_oct(f.g, b, f.b, 1, s, h->scale));
    hipLaunchKernelGGL(k3_sumsq, dim3(nblk(f.g.field)), dim3(256), 0, s, f.g, (const double *)f.b, h->d_part);
    HIP3(hipGetLastError());
    // ||b||'s tag, and one a cycle behind it
    const double tag0 = h->tags.take(1 + (std::uint64_t)std::max(h->prm.max_cycles, 0));
    ST3(reduce_sum(h, h->d_part, (long long)nblk(f.g.field), tag0, s));
    ST3(to_oct(f.g, u, f.x[0], 1, s));
    h->cur = 0;
    double bb = 0.0;
    ST3(wait_sum(h, tag0, s, &bb));
    if (bb != 0.0 && overlapped(h)) {
        ST3(half_sweep(h, h->L - 1, 0, 0, false, 0, s));
        ST3(second_half(h, 0, s));
    }
    const double bn = std::sqrt(bb);
    if (info) {
        std::memset(info, 0, sizeof *info);
        info->levels = h->L;
        info->collapse_level = h->lstar;
        for (int l = 0; l < h->L && l < HIPBMG_MAX_LEVELS; ++l) info->model_us[l] = h->model_us[l];
    }
    hipbmg_status rc = HIPBMG_OK;
    int cycles = 0;
    double rel = 0.0;
    if (bn == 0.0) {
        HIP3(hipMemsetAsync(u, 0, (size_t)f.g.nx * f.g.ny * f.g.nz * sizeof(double), s));
        HIP3(hipStreamSynchronize(s));
    } else {
        rc = HIPBMG_ENOCONV;
        while (cycles < h->prm.max_cycles) {
            ST3(cycle_and_norm(h, s));
            double rr = 0.0;
            ST3(wait_sum(h, tag0 + cycles + 1, s, &rr));
            rel = std::sqrt(rr) / bn;
            if (info) info->relres_hist[cycles] = rel;
            ++cycles;
            if (!std::isfinite(rel)) {
                rc = fail3(HIPBMG_ENAN, "residual norm is not finite after cycle %d", cycles);
                break;
            }
            if (rel <= tol) {
                rc = HIPBMG_OK;
                break;
            }
        }
        ST3(from_oct(f.g, f.x[h->cur], u, s));
        HIP3(hipStreamSynchronize(s));
        if (rc == HIPBMG_ENOCONV) fail3(rc, "tolerance not reached in %d cycles", cycles);
    }
    drain.done = true;   // both ways here have synchronised
    if (h->prof) ST3(prof_collect(h));
    if (info) {
        info->cycles = cycles;
        info->outer_steps = cycles;
        info->relres = rel;
        info->solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    }
    return rc;
}

extern "C" hipbmg_status hipbmg3d_op_smooth(hipbmg3d_handle h, int l, const double *b, double *x, int sweeps,
                                           void *stream)
{
    if (!h || !b || !x) return fail3(HIPBMG_EINVAL, "null argument");
    if (l < 0 || l >= h->L || sweeps < 0) return fail3(HIPBMG_EINVAL, "bad level or sweeps");
    hipStream_t s = (hipStream_t)stream;
    Lev3 &v = h->lv[l];
    ST3(to_oct(v.g, b, v.b, 1, s, h->scale));
    ST3(to_oct(v.g, x, v.x[0], 1, s));
    int cur = 0;
    ST3(relax(h, l, &cur, sweeps, s));
    ST3(from_oct(v.g, v.x[cur], x, s));
    HIP3(hipStreamSynchronize(s));
    h->marks.clear();
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_op_residual(hipbmg3d_handle h, int l, const double *b, const double *x,
                                             double *r, void *stream)
{
    if (!h || !b || !x || !r) return fail3(HIPBMG_EINVAL, "null argument");
    if (l < 0 || l >= h->L) return fail3(HIPBMG_EINVAL, "bad level");
    hipStream_t s = (hipStream_t)stream;
    Lev3 &v = h->lv[l];
    ST3(to_oct(v.g, b, v.b, 1, s, h->scale));
    ST3(to_oct(v.g, x, v.x[0], 1, s));
    ST3(residual(h, l, 0, s));
    ST3(from_oct(v.g, v.r, r, s, 1.0 / h->scale));
    HIP3(hipStreamSynchronize(s));
    h->marks.clear();
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_op_restrict(hipbmg3d_handle h, int l, const double *r, double *bc, void *stream)
{
    if (!h || !r || !bc) return fail3(HIPBMG_EINVAL, "null argument");
    if (l < 1 || l >= h->L) return fail3(HIPBMG_EINVAL, "bad level");
    hipStream_t s = (hipStream_t)stream;
    Lev3 &v = h->lv[l];
    ST3(to_oct(v.g, r, v.r, 1, s));
    ST3(restrict_to(h, l, true, s));
    ST3(from_oct(h->lv[l - 1].g, h->lv[l - 1].b, bc, s));
    HIP3(hipStreamSynchronize(s));
    h->marks.clear();
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_op_interp_correct(hipbmg3d_handle h, int l, double *x, const double *r,
                                                   const double *xc, int rescorr, void *stream)
{
    if (!h || !x || !r || !xc) return fail3(HIPBMG_EINVAL, "null argument");
    if (l < 1 || l >= h->L) return fail3(HIPBMG_EINVAL, "bad level");
    hipStream_t s = (hipStream_t)stream;
    Lev3 &v = h->lv[l];
    ST3(to_oct(v.g, x, v.x[0], 1, s));
    ST3(to_oct(v.g, r, v.r, 1, s, h->scale));
    ST3(to_oct(h->lv[l - 1].g, xc, h->lv[l - 1].x[0], 1, s));
    ST3(interp_from(h, l, 0, 0, rescorr, s));
    ST3(from_oct(v.g, v.x[0], x, s));
    HIP3(hipStreamSynchronize(s));
    h->marks.clear();
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_op_coarse_solve(hipbmg3d_handle h, const double *b, double *x, void *stream)
{
    if (!h || !b || !x) return fail3(HIPBMG_EINVAL, "null argument");
    hipStream_t s = (hipStream_t)stream;
    Lev3 &c = h->lv[0];
    ST3(to_oct(c.g, b, c.b, 1, s, h->scale));
    hipLaunchKernelGGL(k3_fill0, dim3((unsigned)std::min<long long>(nblk(c.g.field), 2048)), dim3(256), 0, s,
                       c.x[0], c.g.field);
    HIP3(hipGetLastError());
    ST3(collapse(h, 0, s));
    ST3(from_oct(c.g, c.x[0], x, s));
    HIP3(hipStreamSynchronize(s));
    h->marks.clear();
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_profile(hipbmg3d_handle h, int enable)
{
    if (!h) return fail3(HIPBMG_EINVAL, "null argument");
    h->prof = enable ? 1 : 0;
    for (int k = 0; k < NPROF3; ++k) {
        h->prof_ms[k] = 0.0;
        h->prof_n[k] = 0.0;
        h->prof_b[k] = 0.0;
    }
    h->marks.clear();
    return HIPBMG_OK;
}

extern "C" hipbmg_status hipbmg3d_profile_read(hipbmg3d_handle h, int k, double *ms_host, long long *launches_host,
                                               double *bytes_per_launch_host)
{
    if (!h) return fail3(HIPBMG_EINVAL, "null argument");
    if (k < 0 || k >= NPROF3) return fail3(HIPBMG_EINVAL, "kernel class %d out of range", k);
    if (ms_host) *ms_host = h->prof_ms[k];
    if (launches_host) *launches_host = (long long)(h->prof_n[k] + 0.5);
    if (bytes_per_launch_host) *bytes_per_launch_host = h->prof_n[k] > 0.0 ? h->prof_b[k] / h->prof_n[k] : 0.0;
    return HIPBMG_OK;
}
