// Streaming vector kernels for the Krylov solver and the tuner.
//
// Reductions are deterministic: a fixed grid of kRedBlocks x kRedThreads
// threads accumulates in FP64 with a grid-stride loop, each block writes one
// partial, and the partials are added in a fixed order.  Scalars (alpha, beta,
// norms) stay on the device between kernels, so a CG iteration needs no host
// round trip.
#include "blas.h"

namespace mfhex {

namespace {

template <typename T>
__device__ __forceinline__ double ld(const T *p, int64_t i) { return (double)p[i]; }

// Sum over the block, in every thread: inside each wavefront by a butterfly, then over the wavefronts in order.
__device__ __forceinline__ double block_sum(double v, double *sh)
{
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
    if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64] = v;
    __syncthreads();
    v = sh[0];
#pragma unroll
    for (int w = 1; w < kRedThreads / 64; ++w) v += sh[w];
    __syncthreads();
    return v;
}

// Sum of a reduction's kRedBlocks partials, in every thread of the block.
__device__ __forceinline__ double partial_sum(const double *partial, double *sh)
{
    double v = 0.0;
#pragma unroll
    for (int i = 0; i < kRedBlocks; i += kRedThreads) v += partial[i + threadIdx.x];
    return block_sum(v, sh);
}

// Grid-stride loop of four entries at a time: load(i, u) for all four before use(i, u).
template <typename Load, typename Use>
__device__ __forceinline__ void stream4(int64_t n, Load load, Use use)
{
    constexpr int64_t S = (int64_t)kRedBlocks * kRedThreads;
    int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x;
    for (; i + 3 * S < n; i += 4 * S) {
#pragma unroll
        for (int u = 0; u < 4; ++u) load(i + u * S, u);
#pragma unroll
        for (int u = 0; u < 4; ++u) use(i + u * S, u);
    }
    for (; i < n; i += S) {
        load(i, 0);
        use(i, 0);
    }
}

__device__ __forceinline__ double block_max(double v, double *sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
#pragma unroll
    for (int s = kRedThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    return sh[0];
}

template <typename TA, typename TB>
__global__ void __launch_bounds__(kRedThreads) k_dot(const TA *__restrict__ a, const TB *__restrict__ b, int64_t n,
                                                     double *__restrict__ partial)
{
    __shared__ double sh[kRedThreads / 64];
    double s = 0.0, u[4], v[4];
    stream4(
        n, [&](int64_t i, int k) { u[k] = ld(a, i), v[k] = ld(b, i); }, [&](int64_t, int k) { s += u[k] * v[k]; });
    s = block_sum(s, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kRedThreads) k_finalize(const double *__restrict__ partial, double *__restrict__ sc,
                                                          int k)
{
    __shared__ double sh[kRedThreads / 64];
    const double s = partial_sum(partial, sh);
    if (threadIdx.x == 0) sc[k] = s;
}

// The scalar steps of an iteration have no launch of their own: each block of the vector kernel that needs alpha or
// beta adds the partials again (8 KB from the L2, in the same order, so all blocks have the same value), and block 0
// writes the scalars.  A slot that block 0 writes is never one that the kernel reads: alpha's kernel saves r.r and
// r.z as the previous ones, which beta's kernel reads.

// beta = (r.r)_new / (r.r)_old, preconditioned (r.z)_new / (r.z)_old; rr, rz and the history by the caller's choice.
struct Beta {
    double rr, rz, beta;
    __device__ __forceinline__ void set(const double *partial, const double *sc, bool pre, double *sh)
    {
        rr = partial_sum(partial, sh);
        rz = pre ? partial_sum(partial + kRedBlocks, sh) : 0.0;
        const double old = sc[pre ? kScRZPrev : kScRRPrev];
        beta = old > 0.0 ? (pre ? rz : rr) / old : 0.0;
    }
    __device__ __forceinline__ void store(double *sc, bool pre, int k, double *hist, int hist_len) const
    {
        sc[kScRRNew] = rr;
        sc[kScRR] = rr;
        sc[kScBeta] = beta;
        if (pre) sc[kScRZ] = rz;
        if (!isfinite(rr) || !isfinite(rz)) sc[kScFlag] = 1.0;
        if (hist && k >= 0 && k < hist_len) hist[k] = sqrt(rr);
    }
};

__global__ void __launch_bounds__(kRedThreads) k_beta(const double *__restrict__ partial, double *__restrict__ sc,
                                                      int pre, int k, double *__restrict__ hist, int hist_len)
{
    __shared__ double sh[kRedThreads / 64];
    Beta b;
    b.set(partial, sc, pre, sh);
    if (threadIdx.x == 0) b.store(sc, pre, k, hist, hist_len);
}

// alpha = r.r / p.Ap (preconditioned: r.z / p.Ap) from the partials of p.Ap; a breakdown gives 0 and sets the flag.
__device__ __forceinline__ double alpha_step(const double *pap, double *sc, bool pre, double *sh)
{
    const double rr = sc[kScRR], rz = sc[kScRZ], s = partial_sum(pap, sh);
    double al = (pre ? rz : rr) / s;
    const bool bad = !(s > 0.0) || !isfinite(al);
    if (bad) al = 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc[kScPAp] = s;
        sc[kScAlpha] = al;
        sc[kScRRPrev] = rr;
        if (pre) sc[kScRZPrev] = rz;
        if (bad) sc[kScFlag] = 1.0;
    }
    return al;
}

// x += alpha p; r -= alpha Ap; partial sums of r.r.  x is FP64; r, p, Ap in T.
// 1e6 nodes, FP64: 48 MB in 7.4 us and 3.5 us of the scalar's own launch before, 7.6 us with it now;
// the iteration's other vector work: dot and its scalars 4.7 + 3.5, update of p 4.7, zero fill 4.9 before, 4.7 and 6.6
// now (30 iterations at p = 5, 1.03e6 nodes: 1752 -> 1495 us).
template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_update_xr(double *__restrict__ x, T *__restrict__ r,
                                                           const T *__restrict__ p, const T *__restrict__ Ap,
                                                           const double *__restrict__ pap, double *sc, int pre,
                                                           int64_t n, double *__restrict__ partial)
{
    __shared__ double sh[kRedThreads / 64];
    const double al = alpha_step(pap, sc, pre, sh);
    double s = 0.0, xi[4];
    T ri[4], pi[4], ai[4];
    stream4(
        n, [&](int64_t i, int k) { xi[k] = x[i], ri[k] = r[i], pi[k] = p[i], ai[k] = Ap[i]; },
        [&](int64_t i, int k) {
            x[i] = xi[k] + al * (double)pi[k];
            const T v = (T)((double)ri[k] - al * (double)ai[k]);
            r[i] = v;
            s += (double)v * (double)v;
        });
    s = block_sum(s, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// x += alpha p; r -= alpha Ap; z = dinv r; partial sums of r.r and r.z.
template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_update_xrz(double *__restrict__ x, T *__restrict__ r,
                                                            const T *__restrict__ p, const T *__restrict__ Ap,
                                                            const T *__restrict__ dinv, T *__restrict__ z,
                                                            const double *__restrict__ pap, double *sc, int64_t n,
                                                            double *__restrict__ partial)
{
    __shared__ double sh[kRedThreads / 64];
    const double al = alpha_step(pap, sc, true, sh);
    double srr = 0.0, srz = 0.0, xi[4];
    T ri[4], pi[4], ai[4], di[4];
    stream4(
        n, [&](int64_t i, int k) { xi[k] = x[i], ri[k] = r[i], pi[k] = p[i], ai[k] = Ap[i], di[k] = dinv[i]; },
        [&](int64_t i, int k) {
            x[i] = xi[k] + al * (double)pi[k];
            const T v = (T)((double)ri[k] - al * (double)ai[k]);
            const T w = (T)((double)di[k] * (double)v);
            r[i] = v;
            z[i] = w;
            srr += (double)v * (double)v;
            srz += (double)v * (double)w;
        });
    srr = block_sum(srr, sh);
    srz = block_sum(srz, sh);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = srr;
        partial[kRedBlocks + blockIdx.x] = srz;
    }
}

// z = dinv r; partial sums of r.z.
template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_precond(const T *__restrict__ r, const T *__restrict__ dinv,
                                                         T *__restrict__ z, int64_t n, double *__restrict__ partial)
{
    __shared__ double sh[kRedThreads / 64];
    double s = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)kRedBlocks * kRedThreads) {
        const T zi = (T)((double)dinv[i] * (double)r[i]);
        z[i] = zi;
        s += (double)r[i] * (double)zi;
    }
    s = block_sum(s, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

__global__ void k_jacobi_inverse(const double *__restrict__ d, double *__restrict__ dinv64, float *__restrict__ dinv32,
                                 int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)kRedBlocks * kRedThreads) {
        const double v = d[i] > 0.0 ? 1.0 / d[i] : 0.0;
        dinv64[i] = v;
        if (dinv32) dinv32[i] = (float)v;
    }
}

// p = r + beta p and, unless null, zero = 0 (the next product's destination).  beta from the partials of r.r (and r.z),
// or with null partials the stored one.
template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_update_p(const T *__restrict__ r, T *__restrict__ p,
                                                          T *__restrict__ zero, const double *__restrict__ partial,
                                                          double *sc, int pre, int k, double *__restrict__ hist,
                                                          int hist_len, int64_t n)
{
    __shared__ double sh[kRedThreads / 64];
    double be;
    if (partial) {
        Beta b;
        b.set(partial, sc, pre, sh);
        if (blockIdx.x == 0 && threadIdx.x == 0) b.store(sc, pre, k, hist, hist_len);
        be = b.beta;
    } else {
        be = sc[kScBeta];
    }
    T ri[4], pi[4];
    stream4(
        n, [&](int64_t i, int u) { ri[u] = r[i], pi[u] = p[i]; },
        [&](int64_t i, int u) {
            p[i] = (T)((double)ri[u] + be * (double)pi[u]);
            if (zero) zero[i] = T(0);
        });
}

// r = b - Ax (Ax may be null: r = b) into r64 and/or r32; partial sums of r.r (FP64 r).
__global__ void __launch_bounds__(kRedThreads) k_residual(const double *__restrict__ b, const double *__restrict__ Ax,
                                                          double *__restrict__ r64, float *__restrict__ r32, int64_t n,
                                                          double *__restrict__ partial)
{
    __shared__ double sh[kRedThreads / 64];
    double s = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)kRedBlocks * kRedThreads) {
        const double ri = Ax ? b[i] - Ax[i] : b[i];
        if (r64) r64[i] = ri;
        if (r32) r32[i] = (float)ri;
        s += ri * ri;
    }
    s = block_sum(s, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

template <typename TS, typename TD>
__global__ void k_copy(const TS *__restrict__ s, TD *__restrict__ d, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)kRedBlocks * kRedThreads)
        d[i] = (TD)s[i];
}

__device__ __forceinline__ uint64_t splitmix64(uint64_t z)
{
    z += 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// Zero fill as a kernel rather than a runtime memset, so that the asynchronous entry points stay
// safe to record into a graph.
// 16-byte stores for the bulk, then the last (bytes mod 16) / 4 words
__global__ void k_zero16(uint4 *__restrict__ p, int64_t n, uint32_t *__restrict__ tail, int ntail)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t i = t; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = make_uint4(0u, 0u, 0u, 0u);
    if (t < ntail) tail[t] = 0u;
}

__global__ void k_zero4(uint32_t *__restrict__ p, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

__global__ void k_fill_uniform(double *__restrict__ x, int64_t n, uint64_t seed)
{
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)kRedBlocks * kRedThreads) {
        const uint64_t z = splitmix64(seed * 0x632be59bd9b4e019ull + (uint64_t)i);
        x[i] = 2.0 * ((double)(z >> 11) * (1.0 / 9007199254740992.0)) - 1.0;
    }
}

template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_maxdiff(const T *__restrict__ a, const T *__restrict__ b, int64_t n,
                                                         double *__restrict__ partial)
{
    __shared__ double sh[kRedThreads];
    double d = 0.0, m = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; i < n; i += (int64_t)kRedBlocks * kRedThreads) {
        const double ai = a[i], bi = b[i];
        d = fmax(d, fabs(ai - bi));
        m = fmax(m, fabs(bi));
        if (ai != ai) d = INFINITY;
    }
    d = block_max(d, sh);
    __syncthreads();
    m = block_max(m, sh);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = d;
        partial[kRedBlocks + blockIdx.x] = m;
    }
}

__global__ void __launch_bounds__(kRedThreads) k_maxfinal(const double *__restrict__ partial, double *__restrict__ out2)
{
    __shared__ double sh[kRedThreads];
    double d = 0.0, m = 0.0;
    for (int i = threadIdx.x; i < kRedBlocks; i += kRedThreads) {
        d = fmax(d, partial[i]);
        m = fmax(m, partial[kRedBlocks + i]);
    }
    d = block_max(d, sh);
    __syncthreads();
    m = block_max(m, sh);
    if (threadIdx.x == 0) {
        out2[0] = d;
        out2[1] = m;
    }
}

}  // namespace

#define GRID dim3(kRedBlocks), dim3(kRedThreads), 0, s

hipError_t launch_dot(const void *a, int pa, const void *b, int pb, int64_t n, double *partial, hipStream_t s)
{
    if (pa == MFHEX_F64 && pb == MFHEX_F64)
        hipLaunchKernelGGL((k_dot<double, double>), GRID, (const double *)a, (const double *)b, n, partial);
    else if (pa == MFHEX_F32 && pb == MFHEX_F32)
        hipLaunchKernelGGL((k_dot<float, float>), GRID, (const float *)a, (const float *)b, n, partial);
    else if (pa == MFHEX_F64)
        hipLaunchKernelGGL((k_dot<double, float>), GRID, (const double *)a, (const float *)b, n, partial);
    else
        hipLaunchKernelGGL((k_dot<float, double>), GRID, (const float *)a, (const double *)b, n, partial);
    return hipGetLastError();
}

hipError_t launch_finalize(const double *partial, double *sc, int k, hipStream_t s)
{
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(kRedThreads), 0, s, partial, sc, k);
    return hipGetLastError();
}

hipError_t launch_beta(const double *partial, double *sc, bool pre, int k, double *hist, int hist_len, hipStream_t s)
{
    hipLaunchKernelGGL(k_beta, dim3(1), dim3(kRedThreads), 0, s, partial, sc, pre ? 1 : 0, k, hist, hist_len);
    return hipGetLastError();
}

hipError_t launch_update_xrz(double *x, void *r, const void *p, const void *Ap, const void *dinv, void *z, int prec,
                             const double *pap, double *sc, int64_t n, double *partial, hipStream_t s)
{
    if (prec == MFHEX_F64)
        hipLaunchKernelGGL(k_update_xrz<double>, GRID, x, (double *)r, (const double *)p, (const double *)Ap,
                           (const double *)dinv, (double *)z, pap, sc, n, partial);
    else
        hipLaunchKernelGGL(k_update_xrz<float>, GRID, x, (float *)r, (const float *)p, (const float *)Ap,
                           (const float *)dinv, (float *)z, pap, sc, n, partial);
    return hipGetLastError();
}

hipError_t launch_precond(const void *r, const void *dinv, void *z, int prec, int64_t n, double *partial,
                          hipStream_t s)
{
    if (prec == MFHEX_F64)
        hipLaunchKernelGGL(k_precond<double>, GRID, (const double *)r, (const double *)dinv, (double *)z, n, partial);
    else
        hipLaunchKernelGGL(k_precond<float>, GRID, (const float *)r, (const float *)dinv, (float *)z, n, partial);
    return hipGetLastError();
}

hipError_t launch_jacobi_inverse(const double *d, double *dinv64, float *dinv32, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_jacobi_inverse, GRID, d, dinv64, dinv32, n);
    return hipGetLastError();
}

hipError_t launch_update_xr(double *x, void *r, const void *p, const void *Ap, int prec, const double *pap, double *sc,
                            bool pre, int64_t n, double *partial, hipStream_t s)
{
    if (prec == MFHEX_F64)
        hipLaunchKernelGGL(k_update_xr<double>, GRID, x, (double *)r, (const double *)p, (const double *)Ap, pap, sc,
                           pre ? 1 : 0, n, partial);
    else
        hipLaunchKernelGGL(k_update_xr<float>, GRID, x, (float *)r, (const float *)p, (const float *)Ap, pap, sc,
                           pre ? 1 : 0, n, partial);
    return hipGetLastError();
}

hipError_t launch_update_p(const void *r, void *p, void *zero, int prec, const double *partial, double *sc, bool pre,
                           int k, double *hist, int hist_len, int64_t n, hipStream_t s)
{
    if (prec == MFHEX_F64)
        hipLaunchKernelGGL(k_update_p<double>, GRID, (const double *)r, (double *)p, (double *)zero, partial, sc,
                           pre ? 1 : 0, k, hist, hist_len, n);
    else
        hipLaunchKernelGGL(k_update_p<float>, GRID, (const float *)r, (float *)p, (float *)zero, partial, sc,
                           pre ? 1 : 0, k, hist, hist_len, n);
    return hipGetLastError();
}

hipError_t launch_residual(const double *b, const double *Ax, double *r64, float *r32, int64_t n, double *partial,
                           hipStream_t s)
{
    hipLaunchKernelGGL(k_residual, GRID, b, Ax, r64, r32, n, partial);
    return hipGetLastError();
}

hipError_t launch_copy(const void *src, int ps, void *dst, int pd, int64_t n, hipStream_t s)
{
    if (ps == MFHEX_F64 && pd == MFHEX_F64)
        hipLaunchKernelGGL((k_copy<double, double>), GRID, (const double *)src, (double *)dst, n);
    else if (ps == MFHEX_F64 && pd == MFHEX_F32)
        hipLaunchKernelGGL((k_copy<double, float>), GRID, (const double *)src, (float *)dst, n);
    else if (ps == MFHEX_F32 && pd == MFHEX_F64)
        hipLaunchKernelGGL((k_copy<float, double>), GRID, (const float *)src, (double *)dst, n);
    else
        hipLaunchKernelGGL((k_copy<float, float>), GRID, (const float *)src, (float *)dst, n);
    return hipGetLastError();
}

hipError_t launch_zero(void *p, size_t bytes, hipStream_t s)
{
    if (bytes % 4) return hipErrorInvalidValue;
    if (bytes == 0) return hipSuccess;
    const bool wide = (uintptr_t)p % 16 == 0;
    const int64_t n = (int64_t)(wide ? bytes / 16 : bytes / 4);
    const int64_t blocks = n < 256 ? 1 : (n + 255) / 256 < 65536 ? (n + 255) / 256 : 65536;
    if (wide)
        hipLaunchKernelGGL(k_zero16, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<uint4 *>(p), n,
                           reinterpret_cast<uint32_t *>(static_cast<char *>(p) + 16 * n), (int)(bytes % 16 / 4));
    else
        hipLaunchKernelGGL(k_zero4, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<uint32_t *>(p), n);
    return hipGetLastError();
}

hipError_t launch_fill_uniform(double *x, int64_t n, uint64_t seed, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_uniform, GRID, x, n, seed);
    return hipGetLastError();
}

hipError_t launch_relmaxdiff(const void *a, const void *b, int64_t n, int prec, double *partial, double *out2,
                             hipStream_t s)
{
    if (prec == MFHEX_F64)
        hipLaunchKernelGGL(k_maxdiff<double>, GRID, (const double *)a, (const double *)b, n, partial);
    else
        hipLaunchKernelGGL(k_maxdiff<float>, GRID, (const float *)a, (const float *)b, n, partial);
    hipLaunchKernelGGL(k_maxfinal, dim3(1), dim3(kRedThreads), 0, s, partial, out2);
    return hipGetLastError();
}

}  // namespace mfhex
