// bmg_dense.hip -- the coarse levels as one dense operator.
//
// On levels 0..d the V-cycle of Algorithm 1 starts from zero, so what it does
// to a right-hand side is linear: x_d = M b_d with a dense matrix M of the
// n = (nx-2)(ny-2) unknowns of level d, whose column c is the V-cycle of the
// unit vector e_c.  A collapsed workgroup walks about 20 dependent barrier
// phases per level, bound by latency whatever the level's size; the product
// is one launch without a single dependent step.  M is formed once per
// hierarchy, in FP64, by the same relaxations, transfers and Cholesky
// substitutions as the collapse, one workgroup per column.
#include "bmg_check.h"

namespace hbmg {

namespace {

// the values of two columns at a vertex
typedef double D2 __attribute__((ext_vector_type(2)));

// a level as a workgroup's two columns see it: operator and weights in global
// memory (every column reads them, so they sit in L2), iterate, residual and
// right-hand side in LDS at compact pitch nx
struct DV {
    int nx, ny, P;
    const double *C, *W, *S, *SW, *SE;
    D2 *x, *r, *b;
    const double *wt;
    int cpitch;
    size_t cplane;
};

__device__ __forceinline__ DV dview(const DenseBuildArgs &a, int l)
{
    extern __shared__ __align__(16) D2 dsm[];
    const LevelDev<double> &g = a.levels[l];
    DV v;
    v.nx = g.nx;
    v.ny = g.ny;
    v.P = g.pitch;
    v.C = g.C;
    v.W = g.W;
    v.S = g.S;
    v.SW = g.SW;
    v.SE = g.SE;
    const int n = g.nx * g.ny;
    v.x = dsm + a.lds_off[l];
    v.r = v.x + n;
    v.b = v.x + 2 * n;
    v.wt = g.wt;
    v.cpitch = g.cpitch;
    v.cplane = g.cplane;
    return v;
}

// residual (b - A x) at interior vertex (i, j)
__device__ __forceinline__ D2 dres(const DV &L, int i, int j, double &diag)
{
    const int P = L.P, n = L.nx, q = j * n + i;
    const size_t p = (size_t)j * P + i;
    const D2 *x = L.x;
    diag = L.C[p];
    const D2 s = L.b[q] + L.W[p] * x[q - 1] + L.W[p + 1] * x[q + 1] + L.S[p] * x[q - n] + L.S[p + P] * x[q + n] +
                     L.SW[p] * x[q - n - 1] + L.SW[p + P + 1] * x[q + n + 1] + L.SE[p] * x[q - n + 1] +
                     L.SE[p + P - 1] * x[q + n - 1];
    return s - diag * x[q];
}

__device__ __forceinline__ void dsweep(const DV &L)
{
    for (int k = 0; k < 4; ++k) {
        const int i0 = (k & 1) ? 1 : 2, j0 = (k >> 1) ? 1 : 2;
        const int ni = L.nx - 2 >= i0 ? (L.nx - 2 - i0) / 2 + 1 : 0, nj = L.ny - 2 >= j0 ? (L.ny - 2 - j0) / 2 + 1 : 0;
        for (int idx = threadIdx.x; idx < ni * nj; idx += blockDim.x) {
            const int jj = idx / ni, i = i0 + 2 * (idx - jj * ni), j = j0 + 2 * jj;
            double d;
            const D2 r = dres(L, i, j, d);
            L.x[j * L.nx + i] += r / d;
        }
        __syncthreads();
    }
}

// b_c = P^T r at the coarse level's interior vertices
__device__ __forceinline__ void drestrict(const DV &F, const DV &Cl)
{
    const int ni = Cl.nx - 2, n = ni * (Cl.ny - 2), P = F.nx, WP = F.cpitch;
    const size_t cp = F.cplane;
    const double *w = F.wt;
    const D2 *r = F.r;
    for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
        const int J = 1 + idx / ni, I = 1 + idx % ni;
        const int f = 2 * J * P + 2 * I;
        const size_t c = (size_t)J * WP + I, cW = c - 1, cS = c - WP, cSW = c - WP - 1;
        Cl.b[J * Cl.nx + I] = r[f] + w[WXL * cp + c] * r[f + 1] + w[WXR * cp + cW] * r[f - 1] +
                              w[WYB * cp + c] * r[f + P] + w[WYT * cp + cS] * r[f - P] +
                              w[WCSW * cp + c] * r[f + P + 1] + w[WCSE * cp + cW] * r[f + P - 1] +
                              w[WCNW * cp + cS] * r[f - P + 1] + w[WCNE * cp + cSW] * r[f - P - 1];
    }
}

// x += P x_c (+ r/C at vertices that are not coarse points)
__device__ __forceinline__ void dinterp(const DV &F, const DV &Cl, int rescorr)
{
    const int ni = F.nx - 2, n = ni * (F.ny - 2), CP = Cl.nx;
    const size_t cp = F.cplane;
    const double *w = F.wt;
    const D2 *xc = Cl.x;
    for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
        const int j = 1 + idx / ni, i = 1 + idx % ni;
        const int c = (j >> 1) * CP + (i >> 1);
        const size_t cw = (size_t)(j >> 1) * F.cpitch + (i >> 1);
        D2 v;
        if (!(i & 1) && !(j & 1)) {
            v = xc[c];
        } else {
            if ((i & 1) && !(j & 1))
                v = w[WXL * cp + cw] * xc[c] + w[WXR * cp + cw] * xc[c + 1];
            else if (!(i & 1) && (j & 1))
                v = w[WYB * cp + cw] * xc[c] + w[WYT * cp + cw] * xc[c + CP];
            else
                v = w[WCSW * cp + cw] * xc[c] + w[WCSE * cp + cw] * xc[c + 1] + w[WCNW * cp + cw] * xc[c + CP] +
                    w[WCNE * cp + cw] * xc[c + CP + 1];
            if (rescorr) v += F.r[j * F.nx + i] / F.C[(size_t)j * F.P + i];
        }
        F.x[j * F.nx + i] += v;
    }
}

}  // namespace

// Columns 2 blockIdx.x and 2 blockIdx.x + 1 of M: the V-cycle of levels top..0
// on e_c.  Bound by the operator's reads from L2 (a column walks the top level
// five times) and the latency of its phases; two columns share the reads and
// write M 16 bytes at a time.  The whole matrix of 961 unknowns (33^2) takes
// 52 us (62 with a column per workgroup), of 1833 (49 x 41) 205 us: 232 with its
// coarse factor of 20 unknowns read from memory, a barrier per unknown.  Rows
// kept in registers over a level's colours change nothing: the iterate's reads
// from LDS and the divisions take the time.
__global__ __launch_bounds__(512) void k_dense_build(DenseBuildArgs a)
{
    extern __shared__ __align__(16) D2 dsm[];
    if (*a.active == 0) return;
    const int col = 2 * blockIdx.x;
    for (int t = threadIdx.x; t < a.lds_elems; t += blockDim.x) dsm[t] = 0.0;
    if (a.lds_chol >= 0)
        for (int t = threadIdx.x; t < a.nc * a.nc; t += blockDim.x)
            reinterpret_cast<double *>(dsm + a.lds_chol)[t] = a.chol[t];
    __syncthreads();
    const DV T = dview(a, a.top);
    const int ni = T.nx - 2, n = ni * (T.ny - 2);
    // ld is even, and its columns from n on are zero (an odd n's column n is this
    // workgroup's second)
    for (int row = blockIdx.x; row < n; row += gridDim.x)
        for (int c = n + (n & 1) + threadIdx.x; c < a.ld; c += blockDim.x) a.M[(size_t)row * a.ld + c] = 0.0;
    if (threadIdx.x < 2 && col + (int)threadIdx.x < n) {
        const int c = col + threadIdx.x;
        T.b[(1 + c / ni) * T.nx + 1 + c % ni][threadIdx.x] = 1.0;
    }
    __syncthreads();
    for (int l = a.top; l >= 1; --l) {
        const DV F = dview(a, l), Cl = dview(a, l - 1);
        for (int s = 0; s < a.nu1; ++s) dsweep(F);
        const int m = F.nx - 2, n = m * (F.ny - 2);
        for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
            const int j = 1 + idx / m, i = 1 + idx % m;
            double d;
            F.r[j * F.nx + i] = dres(F, i, j, d);
        }
        __syncthreads();
        drestrict(F, Cl);
        __syncthreads();
    }
    {   // coarsest level: the Cholesky substitutions, unknown k at the k-th interior vertex
        const DV L0 = dview(a, 0);
        D2 *y = dsm + a.lds_y;
        const int m = L0.nx - 2, nc = a.nc;
        if (a.lds_chol >= 0) {
            // one wave, an unknown per lane, the factor in LDS: the same operations
            // without a barrier and a memory latency per unknown
            if (threadIdx.x < 64) {
                const double *ch = reinterpret_cast<const double *>(dsm + a.lds_chol);
                const int r = threadIdx.x, at = r < nc ? (1 + r / m) * L0.nx + 1 + r % m : 0;
                D2 v = r < nc ? L0.b[at] : D2(0.0);
                for (int k = 0; k < nc; ++k) {
                    const D2 vk = D2{__shfl(v.x, k, 64), __shfl(v.y, k, 64)} / ch[k * nc + k];
                    if (r > k && r < nc) v -= ch[r * nc + k] * vk;
                    if (r == k) v = vk;
                }
                for (int k = nc - 1; k >= 0; --k) {
                    const D2 vk = D2{__shfl(v.x, k, 64), __shfl(v.y, k, 64)} / ch[k * nc + k];
                    if (r < k) v -= ch[k * nc + r] * vk;
                    if (r == k) v = vk;
                }
                if (r < nc) L0.x[at] = v;
            }
            __syncthreads();
        } else {
            for (int k = threadIdx.x; k < nc; k += blockDim.x) y[k] = L0.b[(1 + k / m) * L0.nx + 1 + k % m];
            __syncthreads();
            for (int k = 0; k < nc; ++k) {
                const D2 yk = y[k] / a.chol[(size_t)k * nc + k];
                for (int q = k + 1 + threadIdx.x; q < nc; q += blockDim.x) y[q] -= a.chol[(size_t)q * nc + k] * yk;
                __syncthreads();
                if (threadIdx.x == 0) y[k] = yk;
                __syncthreads();
            }
            for (int k = nc - 1; k >= 0; --k) {
                const D2 xk = y[k] / a.chol[(size_t)k * nc + k];
                for (int q = threadIdx.x; q < k; q += blockDim.x) y[q] -= a.chol[(size_t)k * nc + q] * xk;
                __syncthreads();
                if (threadIdx.x == 0) y[k] = xk;
                __syncthreads();
            }
            for (int k = threadIdx.x; k < nc; k += blockDim.x) L0.x[(1 + k / m) * L0.nx + 1 + k % m] = y[k];
            __syncthreads();
        }
    }
    for (int l = 1; l <= a.top; ++l) {
        const DV F = dview(a, l), Cl = dview(a, l - 1);
        dinterp(F, Cl, a.rescorr);
        __syncthreads();
        for (int s = 0; s < a.nu2; ++s) dsweep(F);
    }
    for (int row = threadIdx.x; row < n; row += blockDim.x)
        *reinterpret_cast<D2 *>(a.M + (size_t)row * a.ld + col) = T.x[(1 + row / ni) * T.nx + 1 + row % ni];
}

hipError_t launch_dense_build(const DenseBuildArgs &a, int n, hipStream_t s)
{
    const int lds = (a.lds_elems + (a.lds_chol >= 0 ? (a.nc * a.nc + 1) / 2 : 0)) * (int)sizeof(D2);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_dense_build),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, DENSE_LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dense_build, dim3((n + 1) / 2), dim3(512), lds, s, a);
    return hipGetLastError();
}

// x = M b at level d, a row of M per wave: every load of a row (16 bytes a
// lane, 1 KB a wave and instruction) goes out before the right-hand side is
// in LDS, so the launch costs one memory round trip and a wave reduction.
// Bound by that latency up to about 1000 unknowns and by M's bytes beyond.
// Measured (gfx950, FP64): 3.9 us for 961 unknowns (33^2, M 7.9 MB), where
// the collapsed workgroup takes 31-38 us for the same levels; 8.4 us for 1833
// (49 x 41, 28 MB), where the level's two kernels and the product for 25 x 21
// below it take 14.9 us.
// The sum's order is fixed; columns n..ld-1 of M and of the staged
// right-hand side are zero.
constexpr int DENSE_ROWS = 4;                // rows (waves) of a workgroup
constexpr int DENSE_PRE = DENSE_MAX / 128;   // a row's loads, all in flight

template <typename T>
__global__ __launch_bounds__(64 * DENSE_ROWS) void k_dense_apply(const double *__restrict__ M, int n, int ld,
                                                                const T *__restrict__ b, T *__restrict__ x, int nx,
                                                                int pitch, const int *active, CheckArgs chk)
{
    __shared__ __align__(16) double bs[DENSE_MAX];
    if ((int)blockIdx.x * DENSE_ROWS >= n) {   // the extra workgroup
        cycle_check(chk);
        return;
    }
    if (active && *active == 0) return;
    const int lane = threadIdx.x & 63, row = blockIdx.x * DENSE_ROWS + (threadIdx.x >> 6);
    const int nch = ld >> 7, mine = row < n ? row : n - 1;
    const double2 *m = reinterpret_cast<const double2 *>(M + (size_t)mine * ld) + lane;
    double2 v[DENSE_PRE];
#pragma unroll
    for (int c = 0; c < DENSE_PRE; ++c) v[c] = c < nch ? m[c * 64] : double2{0.0, 0.0};
    const int ni = nx - 2;
    for (int idx = threadIdx.x; idx < ld; idx += 64 * DENSE_ROWS) {
        const int jj = idx / ni;
        bs[idx] = idx < n ? (double)b[(size_t)(1 + jj) * pitch + 1 + idx - jj * ni] : 0.0;
    }
    __syncthreads();
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int c = 0; c < DENSE_PRE; ++c)
        if (c < nch) {
            const double2 q = reinterpret_cast<const double2 *>(bs)[c * 64 + lane];
            s0 += v[c].x * q.x;
            s1 += v[c].y * q.y;
        }
    double s = s0 + s1;
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0 && row < n) {
        const int jj = row / ni;
        x[(size_t)(1 + jj) * pitch + 1 + row - jj * ni] = (T)s;
    }
}

template <typename T>
hipError_t launch_dense_apply(const double *M, int n, int ld, const LevelDev<T> &lv, int xb, const int *active,
                              hipStream_t s, const CheckArgs *chk)
{
    static_assert(64 * DENSE_ROWS >= 256, "cycle_check needs 256 threads");
    const int extra = chk && chk->partials ? 1 : 0;
    hipLaunchKernelGGL((k_dense_apply<T>), dim3((n + DENSE_ROWS - 1) / DENSE_ROWS + extra), dim3(64 * DENSE_ROWS), 0,
                       s, M, n, ld, lv.b, lv.x[xb], lv.nx, lv.pitch, extra ? chk->before() : active,
                       extra ? *chk : CheckArgs{});
    return hipGetLastError();
}
template hipError_t launch_dense_apply<double>(const double *, int, int, const LevelDev<double> &, int, const int *,
                                               hipStream_t, const CheckArgs *);
template hipError_t launch_dense_apply<float>(const double *, int, int, const LevelDev<float> &, int, const int *,
                                              hipStream_t, const CheckArgs *);

}  // namespace hbmg
