// p-multigrid transfer and smoother kernels.
//
// Prolongation P maps a coarse field to its values at the fine nodes: in
// every element the coarse nodal values are interpolated to the fine
// Gauss-Lobatto nodes by the tensor product of the 1D interpolation matrix
// I1 [P_f][P_c] (three 1D contractions, sum factorization as in Sec. 1).  A
// fine node on a face has the same value in each element that shares it, so
// one of them, the last, adds it: no atomics.  The restriction adds
// I1^T (w r_f) per element with weight w = 1/m of the m elements at a node,
// which is exactly P^T r_f; r_f = b - A x is formed as it is read.  m is known
// from the node's position on the structured mesh (2 per direction in which it
// lies on a face between two elements).  Masked (Dirichlet) nodes are skipped
// on both levels.
#include "blas.h"
#include "mg.h"

namespace mfhex {

namespace {

constexpr int kTransferThreads = 128;

// Weight 1/m of local node (i, j, k) of element (ex, ey, ez) with P nodes per direction (a power of 1/2).
template <typename T>
__device__ __forceinline__ T share_weight(int i, int j, int k, int P, int ex, int ey, int ez, int nex, int ney, int nez)
{
    const bool sx = (i == 0 && ex > 0) || (i == P - 1 && ex < nex - 1);
    const bool sy = (j == 0 && ey > 0) || (j == P - 1 && ey < ney - 1);
    const bool sz = (k == 0 && ez > 0) || (k == P - 1 && ez < nez - 1);
    return (sx ? T(0.5) : T(1)) * (sy ? T(0.5) : T(1)) * (sz ? T(0.5) : T(1));
}

// Bound by the chain of its stages (four barriers, two indirect accesses): the destinations' entries are loaded before
// the first stage.  4096 elements from p = 7 to 3: prolongation 24.5 us with atomics, 19.9 without, 17.6 with the early
// loads; restriction 11.7 us and 9 for the residual's own pass before, 16.4 now.
template <int PF, int PC, int DIR, typename T>
__global__ void __launch_bounds__(kTransferThreads)
k_transfer(int nex, int ney, int nez, const int32_t *__restrict__ off_f, const int32_t *__restrict__ off_c,
           const T *__restrict__ I1, const T *__restrict__ src, const T *__restrict__ src2, T *__restrict__ dst,
           T *__restrict__ zero, int64_t nzero)
{
    constexpr int NT = kTransferThreads;
    constexpr int F3 = PF * PF * PF, C3 = PC * PC * PC;
    // DIR 0 (prolong): a = coarse [k][j][i] -> b [k][j][I] -> c [k][J][I] -> fine [K][J][I]
    // DIR 1 (restrict): a = fine [K][J][I] -> b [K][J][i] -> c [K][j][i] -> coarse [k][j][i]
    constexpr int NA = DIR == 0 ? C3 : F3;
    constexpr int NB = DIR == 0 ? PC * PC * PF : PF * PF * PC;
    constexpr int NC = DIR == 0 ? PC * PF * PF : PF * PC * PC;
    __shared__ T sI[PF * PC], sa[NA], sb[NB], sc[NC];
    const int tid = threadIdx.x;
    const int64_t e = blockIdx.x;
    for (int64_t t = e * NT + tid; t < nzero; t += (int64_t)gridDim.x * NT) zero[t] = T(0);
    const int ex = (int)(e % nex), ey = (int)((e / nex) % ney), ez = (int)(e / ((int64_t)nex * ney));
    for (int t = tid; t < PF * PC; t += NT) sI[t] = I1[t];
    constexpr int NOUT = DIR == 0 ? F3 : C3, RO = (NOUT + NT - 1) / NT;
    int32_t od[RO];  // destinations (prolongation: of the nodes that this element owns)
    T xd[RO];
#pragma unroll
    for (int r = 0; r < RO; ++r) {
        const int t = tid + r * NT;
        od[r] = -1;
        if (t < NOUT) {
            if constexpr (DIR == 0) {
                const int i = t % PF, j = (t / PF) % PF, k = t / (PF * PF);
                if ((i < PF - 1 || ex == nex - 1) && (j < PF - 1 || ey == ney - 1) && (k < PF - 1 || ez == nez - 1))
                    od[r] = off_f[e * F3 + t];
            } else {
                od[r] = off_c[e * C3 + t];
            }
        }
    }
    if constexpr (DIR == 0) {
#pragma unroll
        for (int r = 0; r < RO; ++r) xd[r] = od[r] >= 0 ? dst[od[r]] : T(0);
        for (int t = tid; t < C3; t += NT) {
            const int32_t o = off_c[e * C3 + t];
            sa[t] = o >= 0 ? src[o] : T(0);
        }
    } else {
        for (int t = tid; t < F3; t += NT) {
            const int32_t o = off_f[e * F3 + t];
            const int i = t % PF, j = (t / PF) % PF, k = t / (PF * PF);
            sa[t] = o >= 0 ? share_weight<T>(i, j, k, PF, ex, ey, ez, nex, ney, nez) * (src[o] - src2[o])
                           : T(0);
        }
    }
    __syncthreads();
    // x: DIR 0: b[k][j][I] = sum_i I[I][i] a[k][j][i];  DIR 1: b[K][J][i] = sum_I I[I][i] a[K][J][I]
    constexpr int NIX = DIR == 0 ? PC : PF, NOX = DIR == 0 ? PF : PC;
    for (int t = tid; t < NB; t += NT) {
        const int o = t % NOX, rest = t / NOX;
        T s = T(0);
        for (int i = 0; i < NIX; ++i)
            s += (DIR == 0 ? sI[o * PC + i] : sI[i * PC + o]) * sa[i + NIX * rest];
        sb[t] = s;
    }
    __syncthreads();
    // y: contract the middle index
    constexpr int NX = NOX;                     // extent of the (already contracted) fastest index
    constexpr int NIY = DIR == 0 ? PC : PF, NOY = DIR == 0 ? PF : PC;
    for (int t = tid; t < NC; t += NT) {
        const int a = t % NX, o = (t / NX) % NOY, z = t / (NX * NOY);
        T s = T(0);
        for (int j = 0; j < NIY; ++j)
            s += (DIR == 0 ? sI[o * PC + j] : sI[j * PC + o]) * sb[a + NX * (j + NIY * z)];
        sc[t] = s;
    }
    __syncthreads();
    // z: contract the slowest index and add to the destination
    constexpr int NIZ = DIR == 0 ? PC : PF, NOZ = DIR == 0 ? PF : PC, NXY = NX * NOY;
    static_assert(NOZ * NXY == NOUT, "one result per destination");
#pragma unroll
    for (int r = 0; r < RO; ++r) {
        const int t = tid + r * NT;
        if (t >= NOUT || od[r] < 0) continue;
        const int ab = t % NXY, o = t / NXY;
        T s = T(0);
        for (int k = 0; k < NIZ; ++k) s += (DIR == 0 ? sI[o * PC + k] : sI[k * PC + o]) * sc[ab + NXY * k];
        if constexpr (DIR == 0) dst[od[r]] = xd[r] + s;
        else unsafeAtomicAdd(&dst[od[r]], s);
    }
}

template <int PF, int PC, typename T>
hipError_t transfer_t(const TransferLaunch &t)
{
    const int64_t nelem = (int64_t)t.nex * t.ney * t.nez;
    const T *I1 = static_cast<const T *>(t.I1), *src = static_cast<const T *>(t.src);
    const T *src2 = static_cast<const T *>(t.src2);
    T *dst = static_cast<T *>(t.dst), *zero = static_cast<T *>(t.zero);
    if (t.dir == 0)
        hipLaunchKernelGGL((k_transfer<PF, PC, 0, T>), dim3((unsigned)nelem), dim3(kTransferThreads), 0, t.stream,
                           t.nex, t.ney, t.nez, t.off_f, t.off_c, I1, src, src2, dst, zero, t.nzero);
    else
        hipLaunchKernelGGL((k_transfer<PF, PC, 1, T>), dim3((unsigned)nelem), dim3(kTransferThreads), 0, t.stream,
                           t.nex, t.ney, t.nez, t.off_f, t.off_c, I1, src, src2, dst, zero, t.nzero);
    return hipGetLastError();
}

template <int PF, int PC>
hipError_t transfer_pf(const TransferLaunch &t)
{
    return t.prec == MFHEX_F32 ? transfer_t<PF, PC, float>(t) : transfer_t<PF, PC, double>(t);
}

#define GRID dim3(kRedBlocks), dim3(kRedThreads), 0, s

// The smoother's vector steps, one launch between two products.  They also clear what the next launches add into (Ad,
// and at the end of the pre-smoothing the coarse right-hand side), and the step after the last product applies both of
// the directions that are left, so that a smoothing of degree k has k launches besides its products (with a fill for
// each product, x = 0 and the last addition apart it had 2 k + 1, of 4 to 6 us each).
template <typename T>
struct ChebZero {
    T *a;        // Ad
    T *b;        // the coarse right-hand side (nb entries, fewer than n) or null
    int64_t nb;
    __device__ __forceinline__ void at(int64_t i) const
    {
        if (a) a[i] = T(0);
        if (b && i < nb) b[i] = T(0);
    }
};

template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_cheb_init(const T *__restrict__ b, const T *Ax,
                                                           const T *__restrict__ dinv, T *__restrict__ x,
                                                           T *__restrict__ r, T *__restrict__ d, T inv_theta, int zero_x,
                                                           int last, ChebZero<T> z, int64_t n)
{
    const int64_t S = (int64_t)gridDim.x * kRedThreads;
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += S) {
        const T ri = dinv[i] * (Ax ? b[i] - Ax[i] : b[i]), di = ri * inv_theta;
        if (last) {
            x[i] = zero_x ? di : x[i] + di;
        } else {
            r[i] = ri;
            d[i] = di;
        }
        z.at(i);
    }
}

template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_cheb_step(T *__restrict__ x, T *__restrict__ d, T *__restrict__ r,
                                                           const T *Ad, const T *__restrict__ dinv, T cd, T cr,
                                                           int zero_x, int last, ChebZero<T> z, int64_t n)
{
    const int64_t S = (int64_t)gridDim.x * kRedThreads;
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += S) {
        const T di = d[i], ri = r[i] - dinv[i] * Ad[i], dn = cd * di + cr * ri, xi = zero_x ? di : x[i] + di;
        if (last) {
            x[i] = xi + dn;
        } else {
            x[i] = xi;
            r[i] = ri;
            d[i] = dn;
        }
        z.at(i);
    }
}

__global__ void k_mask_scale(double *__restrict__ v, const double *__restrict__ dinv, double scale, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)kRedBlocks * kRedThreads)
        v[i] = dinv[i] > 0.0 ? (scale != 0.0 ? v[i] * scale : v[i]) : 0.0;
}

__global__ void k_scale_by(const double *__restrict__ a, const double *__restrict__ dinv, double *__restrict__ out,
                           int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)kRedBlocks * kRedThreads)
        out[i] = dinv[i] * a[i];
}

__global__ void __launch_bounds__(kRedThreads) k_dot_dinv(const double *__restrict__ v, const double *__restrict__ dinv,
                                                          int64_t n, double *__restrict__ partial)
{
    __shared__ double sh[kRedThreads];
    double s = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)kRedBlocks * kRedThreads)
        if (dinv[i] > 0.0) s += v[i] * v[i] / dinv[i];
    sh[threadIdx.x] = s;
    __syncthreads();
#pragma unroll
    for (int st = kRedThreads / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

}  // namespace

hipError_t launch_transfer(const TransferLaunch &t)
{
    // coarse order max(1, pf / 2)
    switch (t.pf) {
    case 2: return t.pc == 1 ? transfer_pf<3, 2>(t) : hipErrorInvalidValue;
    case 3: return t.pc == 1 ? transfer_pf<4, 2>(t) : hipErrorInvalidValue;
    case 4: return t.pc == 2 ? transfer_pf<5, 3>(t) : hipErrorInvalidValue;
    case 5: return t.pc == 2 ? transfer_pf<6, 3>(t) : hipErrorInvalidValue;
    case 6: return t.pc == 3 ? transfer_pf<7, 4>(t) : hipErrorInvalidValue;
    case 7: return t.pc == 3 ? transfer_pf<8, 4>(t) : hipErrorInvalidValue;
    case 8: return t.pc == 4 ? transfer_pf<9, 5>(t) : hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

// Blocks of a smoother step: one entry a thread as far as 2048 blocks go (eight for each CU).
static dim3 cheb_grid(int64_t n)
{
    const int64_t b = (n + kRedThreads - 1) / kRedThreads;
    return dim3((unsigned)(b < 2048 ? b : 2048));
}

template <typename T>
static hipError_t cheb_init_t(const ChebLaunch &c, const void *Ax, double inv_theta)
{
    const ChebZero<T> z{(T *)c.zero_ad, (T *)c.zero_b, c.nb};
    hipLaunchKernelGGL(k_cheb_init<T>, cheb_grid(c.n), dim3(kRedThreads), 0, c.stream, (const T *)c.b, (const T *)Ax,
                       (const T *)c.dinv, (T *)c.x, (T *)c.r, (T *)c.d, (T)inv_theta, c.zero_x, c.last, z, c.n);
    return hipGetLastError();
}

template <typename T>
static hipError_t cheb_step_t(const ChebLaunch &c, const void *Ad, double cd, double cr)
{
    const ChebZero<T> z{(T *)c.zero_ad, (T *)c.zero_b, c.nb};
    hipLaunchKernelGGL(k_cheb_step<T>, cheb_grid(c.n), dim3(kRedThreads), 0, c.stream, (T *)c.x, (T *)c.d, (T *)c.r,
                       (const T *)Ad, (const T *)c.dinv, (T)cd, (T)cr, c.zero_x, c.last, z, c.n);
    return hipGetLastError();
}

hipError_t launch_cheb_init(const ChebLaunch &c, const void *Ax, double inv_theta)
{
    return c.prec == MFHEX_F32 ? cheb_init_t<float>(c, Ax, inv_theta) : cheb_init_t<double>(c, Ax, inv_theta);
}

hipError_t launch_cheb_step(const ChebLaunch &c, const void *Ad, double cd, double cr)
{
    return c.prec == MFHEX_F32 ? cheb_step_t<float>(c, Ad, cd, cr) : cheb_step_t<double>(c, Ad, cd, cr);
}

hipError_t launch_mask_scale(double *v, const double *dinv, double scale, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_mask_scale, GRID, v, dinv, scale, n);
    return hipGetLastError();
}

hipError_t launch_scale_by(const double *a, const double *dinv, double *out, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_scale_by, GRID, a, dinv, out, n);
    return hipGetLastError();
}

hipError_t launch_dot_dinv(const double *v, const double *dinv, int64_t n, double *partial, hipStream_t s)
{
    hipLaunchKernelGGL(k_dot_dinv, GRID, v, dinv, n, partial);
    return hipGetLastError();
}

}  // namespace mfhex
