// Line-fused operator kernel: the whole element operator in five register stages.
//
// Every stage owns whole lines of an element in registers and does all the
// work that needs only that line before it goes back to LDS:
//   Y    gather an y-line of nodes straight from x; B and D^B along y
//        (D^B = l_i'(x_a), the basis derivative at the points)
//   X    B and D^B along x
//   Z    B and D^B along z: the reference gradient of a z-line of points is
//        now in registers; the pointwise factors act there, and the transposed
//        z contraction follows from the same registers
//   X^T, Y^T  the transposed contractions; the element values of an y-line of
//        nodes leave Y^T in registers, straight into the scatter
// With Gauss-Lobatto points at the nodes B is the identity: Y forms d/ds, X
// d/dr, Z d/dt, then the same way back.  The mass operator carries one array
// through the same stages.  Four barriers an element, and a fifth before the next one
// of a march, instead of thirteen, and 15-17 LDS accesses a point instead of about 26 (Gauss).
//
// Pointwise stage: no stored factors.  The map is trilinear, so along a z-line (r, s fixed) the
// Jacobian columns are j_r, j_s linear in t and j_t constant: a lane forms them
// once per line from the element's seven trilinear coefficients and evaluates
// v = (w / detJ) adj(J) adj(J)^T u from cross products, about 55 FP64
// operations a point in place of 48 bytes of HBM (in FP64 also when x and y
// are FP32: the same result as factors rounded to FP32, or closer).
//
// A thread group owns G elements consecutive in x and marches along y: the
// y-face shared by consecutive elements is carried in registers (one load and
// one atomic fewer per line), the next element's x lines and vertices load
// behind the transposed stages.  Node numbers and Dirichlet masks follow from
// the position in the structured mesh, so no restriction offsets are read.
//
// Measured on MI355X, about 1e7 nodes, FP64, us an apply with its output fill, stored-factor kernel
// (k_apply / k_mass, the best variant) -> this kernel: BP3 p = 1..8 2610 -> 1725, 720 -> 446, 474 -> 258,
// 383 -> 232, 334 -> 208, 287 -> 178, 294 -> 183, 270 -> 198; BP1 p = 3..8 198 -> 143, 200 -> 127,
// 152 -> 127, 168 -> 118, 166 -> 124, 160 -> 129.  HBM traffic is within 1.45 of x and y (p = 3: 90 MB
// read, 135 MB written); the vector units are busy 63% of the time (p = 3) and bound it: about 109 FP64
// operations a point at p = 3, 55 of them geometry.  (Coefficients read from a table of 168 bytes an
// element instead of formed from the vertices gained nothing: 253 us at p = 3.)
#pragma once

#include <type_traits>
#include <utility>

#include "geom.hpp"
#include "mfhex_internal.h"

namespace mfhex {

// The 1D matrices are read through the scalar cache: constant address space, uniform addresses.
template <typename T>
using cptr = const __attribute__((address_space(4))) T *;

template <typename T>
using gptr = __attribute__((address_space(1))) T *;
__device__ __forceinline__ void global_add(gptr<double> p, double v) { __builtin_amdgcn_global_atomic_fadd_f64(p, v); }
__device__ __forceinline__ void global_add(gptr<float> p, float v) { __builtin_amdgcn_global_atomic_fadd_f32(p, v); }

// Keeps the loads of one stage from being hoisted out of the march (there are more coefficients
// than scalar registers).
template <typename T>
__device__ __forceinline__ cptr<T> opaque(cptr<T> p)
{
    asm volatile("" : "+s"(p));
    return p;
}

// Orders the coefficient loads of a row behind a value of an earlier row, so that at most two rows are in flight:
// issued all at once they would not fit the scalar registers (used where the matrices exceed them).
template <typename T>
__device__ __forceinline__ cptr<T> after(cptr<T> p, const T &v)
{
    asm volatile("" : "+s"(p) : "v"(v));
    return p;
}
constexpr bool rows_in_flight(int NI, int NO, int bytes)
{
    // (NI == NO: the collocated derivative, the only matrix of its kernel; else B and the derivative)
    return (NI == NO ? 1 : 2) * ((NO + 1) / 2) * NI * bytes > 240;
}

// A line of N values, folded: e_i = v_i + v_{N-1-i}, d_i = v_i - v_{N-1-i} (i < N/2), e_{N/2} = the middle value.
template <int N, typename T>
struct Folded {
    static constexpr int H = N / 2, MID = N & 1;
    T e[H + MID];
    T d[H > 0 ? H : 1];
    __device__ __forceinline__ void set(const T (&v)[N])
    {
#pragma unroll
        for (int i = 0; i < H; ++i) {
            e[i] = v[i] + v[N - 1 - i];
            d[i] = v[i] - v[N - 1 - i];
        }
        if constexpr (MID) e[H] = v[H];
    }
};

// Even and odd half of the output pair (o, NO-1-o) of a contraction of a folded line: the outputs are E + O and, for
// SYM +1 (M[NO-1-o][NI-1-i] = M[o][i]), E - O, for SYM -1 (M[NO-1-o][NI-1-i] = -M[o][i]) O - E.
template <int NI, int NO, int SYM, typename T>
__device__ __forceinline__ void line_pair(cptr<T> M, const Folded<NI, T> &f, int o, T &E, T &O)
{
    constexpr int H = NI / 2;
    const cptr<T> row = M + o * NI;
    E = T(0), O = T(0);
    const bool middle = 2 * o + 1 == NO;  // one output: only its even (SYM +1) or odd (-1) half is non-zero
#pragma unroll
    for (int i = 0; i < H; ++i) {
        if (!middle || SYM > 0) E += row[i] * f.e[i];
        if (!middle || SYM < 0) O += row[H + i] * f.d[i];
    }
    if constexpr (NI & 1)
        if (!middle || SYM > 0) E += row[2 * H] * f.e[H];
}

// All output pairs of a contraction: put(o, E, O, E + O).
template <int NI, int NO, int SYM, typename T, typename Put>
__device__ __forceinline__ void line_halves(cptr<T> M, const Folded<NI, T> &f, Put put)
{
    constexpr bool TIE = rows_in_flight(NI, NO, sizeof(T));
    if (TIE) M = after<T>(M, f.e[0]);
    cptr<T> cur = M, next = M;
#pragma unroll
    for (int o = 0; o < (NO + 1) / 2; ++o) {
        T E, O;
        line_pair<NI, NO, SYM>(cur, f, o, E, O);
        cur = next;
        T lo = E + O;
        if (TIE) next = after<T>(M, lo);
        put(o, E, O, lo);
    }
}

// The same as put(o, lo, hi) of the outputs o and NO-1-o.
template <int NI, int NO, int SYM, typename T, typename Put>
__device__ __forceinline__ void line_all(cptr<T> M, const Folded<NI, T> &f, Put put)
{
    line_halves<NI, NO, SYM>(M, f, [&](int o, T E, T O, T lo) { put(o, lo, SYM > 0 ? E - O : O - E); });
}

// Transposed contraction of a line of NO values with the same folded rows, accumulated over several matrices:
// out_i = S_i + D_i, out_{NI-1-i} = S_i - D_i.
template <int NI, typename T>
struct TransAcc {
    static constexpr int H = NI / 2, MID = NI & 1;
    T S[H + MID], D[H > 0 ? H : 1];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int i = 0; i < H + MID; ++i) S[i] = T(0);
#pragma unroll
        for (int i = 0; i < H; ++i) D[i] = T(0);
    }
    template <int NO, int SYM>
    __device__ __forceinline__ void add(cptr<T> M, const T (&w)[NO])
    {
        constexpr bool TIE = rows_in_flight(NI, NO, sizeof(T));
        if (TIE) M = after<T>(M, w[0]);
        cptr<T> cur = M, next = M;
#pragma unroll
        for (int o = 0; o < NO / 2; ++o) {
            const T e = w[o] + w[NO - 1 - o], d = w[o] - w[NO - 1 - o];
            const T s = SYM > 0 ? e : d, t = SYM > 0 ? d : e;
            const cptr<T> row = cur + o * NI;
#pragma unroll
            for (int i = 0; i < H; ++i) {
                S[i] += row[i] * s;
                D[i] += row[H + i] * t;
            }
            if constexpr (MID) S[H] += row[2 * H] * s;
            cur = next;
            if (TIE) {
                // (every accumulator: a chain of one of them alone could run ahead of the others)
#pragma unroll
                for (int i = 0; i < H; ++i) asm volatile("" : "+v"(S[i]), "+v"(D[i]));
                next = after<T>(M, S[0]);
            }
        }
        if constexpr (NO & 1) {
            const T m = w[NO / 2];
            const cptr<T> row = cur + (NO / 2) * NI;
#pragma unroll
            for (int i = 0; i < H; ++i) {
                if (SYM > 0) S[i] += row[i] * m;
                else D[i] += row[H + i] * m;
            }
            if constexpr (MID && SYM > 0) S[H] += row[2 * H] * m;
        }
    }
    __device__ __forceinline__ T out(int i) const
    {
        return MID && i == H ? S[H] : i < H ? S[i] + D[i] : S[NI - 1 - i] - D[NI - 1 - i];
    }
};

template <int N, int ST, typename T>
__device__ __forceinline__ void line_read(const T *src, T (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = src[i * ST];
}

// Jacobian columns along the z-line (r, s): jr = jr0 + t jr1, js = js0 + t js1, jt constant.
struct ZLineGeom {
    double jr0[3], jr1[3], js0[3], js1[3], jt[3];

    __device__ __forceinline__ void set(const double *c, double r, double s)
    {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            jr0[d] = c[d] + s * c[6 + d];          // r, rs
            jr1[d] = c[12 + d] + s * c[18 + d];    // rt, rst
            js0[d] = c[3 + d] + r * c[6 + d];      // s, rs
            js1[d] = c[15 + d] + r * c[18 + d];    // st, rst
            jt[d] = c[9 + d] + r * c[12 + d] + s * js1[d];
            // one component's coefficients in registers at a time
            asm volatile("" : "+v"(jr0[d]), "+v"(jr1[d]), "+v"(js0[d]), "+v"(js1[d]), "+v"(jt[d]), "+v"(r));
        }
    }
    // pins the evaluation order: nothing that uses the columns moves above this point
    __device__ __forceinline__ void pin()
    {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            asm volatile("" : "+v"(jr0[d]), "+v"(jr1[d]), "+v"(js0[d]), "+v"(js1[d]), "+v"(jt[d]));
        }
    }
    __device__ __forceinline__ void columns(double t, double jr[3], double js[3]) const
    {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            jr[d] = jr0[d] + t * jr1[d];
            js[d] = js0[d] + t * js1[d];
        }
    }
    // detJ along the line: d[0] + t (d[1] + t d[2])
    __device__ __forceinline__ void det_poly(double d[3]) const
    {
        double a[3], b[3];
        cross(jr0, js0, a);
        d[0] = dot3(jt, a);
        cross(jr1, js1, a);
        d[2] = dot3(jt, a);
        cross(jr0, js1, a);
        cross(jr1, js0, b);
        d[1] = dot3(jt, a) + dot3(jt, b);
    }
};

// 1 / d by the hardware estimate and two Newton steps (relative error about one unit in the last place).
__device__ __forceinline__ double fast_rcp(double d)
{
    double y = __builtin_amdgcn_rcp(d);
    y = fma(fma(-d, y, 1.0), y, y);
    return fma(fma(-d, y, 1.0), y, y);
}

// v = w adj(J) adj(J)^T u / detJ at parameter t of the line.  With the adjugate rows js x jt, jt x jr and jr x js,
//   q = adj(J)^T u = jt x (us jr - ur js) + ut (jr x js),
//   v = (js . (jt x q), -jr . (jt x q), (jr x js) . q) w / detJ,
// which needs no more than the columns and one cross product at a time in registers.
__device__ __forceinline__ void apply_geom(const ZLineGeom &g, double t, double w, double &ur, double &us, double &ut)
{
    double jr[3], js[3], r2[3], h[3], q[3];
    g.columns(t, jr, js);
    cross(jr, js, r2);
    const double f = w * fast_rcp(dot3(g.jt, r2));
#pragma unroll
    for (int d = 0; d < 3; ++d) h[d] = us * jr[d] - ur * js[d];
    cross(g.jt, h, q);
#pragma unroll
    for (int d = 0; d < 3; ++d) q[d] = f * (q[d] + ut * r2[d]);
    cross(g.jt, q, h);
    ur = dot3(js, h);
    us = -dot3(jr, h);
    ut = dot3(r2, q);
}

// LDS of one element: arrays [k][b][a] of P planes of Q rows of PITCH entries.
template <int P, int Q>
struct LineLds {
    static constexpr int PITCH = (Q % 2 == 0) ? Q + 1 : Q;
    static constexpr int PLANE = PITCH * Q;
    static constexpr int ELEM = P * PLANE;
};
constexpr int line_arrays(int mode) { return mode == kMass ? 1 : 3; }
// Entries of the contraction arrays, up to the FP64 tables behind them: whole doubles (in FP32 with q and G odd the
// arrays of the collocated operator end in the middle of one).
template <int P, int Q, typename T>
constexpr int line_array_len(int mode, int G)
{
    constexpr int M = 8 / sizeof(T);
    return (line_arrays(mode) * G * LineLds<P, Q>::ELEM + M - 1) / M * M;
}
template <int P, int Q, typename T>
constexpr size_t line_lds(int mode, int G)
{
    return (size_t)line_array_len<P, Q, T>(mode, G) * sizeof(T) + ((size_t)G * kTriCoef + 2 * Q + 12 * (G + 1)) * 8;
}

// Wavefronts per SIMD that the registers are allocated for: the pointwise stage holds the gradient of a z-line
// (6 Q registers), the columns (30) and one point's work (about 30); four wavefronts (128 registers) fit it up to
// q = 6 without spills, three (168) above.  (Two at q = 5: 283 against 277 us at p = 3, 1e7 nodes.)
constexpr int line_waves(int Q, int mode) { return mode == kDiff && Q > 6 ? 3 : 4; }

template <typename T>
struct LineArgs {
    const T *bas;
    const double *bas64;
    const double *vert, *kappa;
    const T *qdata, *x;  // qdata: stored factors (k_mline)
    T *y, *ebuf;
    int nex, ney, nez, dirichlet, nvec;
    int ngx, nych, march;  // element groups per row, y-chunks per column, elements per march
    unsigned base;         // first thread group of this launch
};

// Marching position of a thread group.
struct LinePos {
    int ex0, nvalid, ey0, ey1, ez;
};
template <int G, typename A>
__device__ __forceinline__ LinePos line_pos_of(const A &a, unsigned bid, unsigned nb)
{
    // XCD x (blocks are dealt round-robin) takes the x-th contiguous range of the groups
    const unsigned xcd = bid % kNumXcd, nq = nb / kNumXcd, nr = nb % kNumXcd;
    const unsigned b = a.base + xcd * nq + (xcd < nr ? xcd : nr) + bid / kNumXcd;
    LinePos q;
    const int gx = (int)(b % (unsigned)a.ngx);
    const unsigned r = b / (unsigned)a.ngx;
    q.ex0 = gx * G;
    q.nvalid = a.nex - q.ex0 < G ? a.nex - q.ex0 : G;
    q.ey0 = (int)(r % (unsigned)a.nych) * a.march;
    q.ey1 = q.ey0 + a.march < a.ney ? q.ey0 + a.march : a.ney;
    q.ez = (int)(r / (unsigned)a.nych);
    return q;
}

template <int P, int Q, bool COLLOC, int MODE, bool VARK, typename T, int G, int NT, bool DET, typename OFF>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(line_waves(Q, MODE))))
k_line(const LineArgs<T> a)
{
    static_assert(!(COLLOC && MODE == kMass), "the collocated mass operator has no contractions");
    using L = LineLds<P, Q>;
    constexpr int p = P - 1, W = G * p + 1, Q2 = Q * Q, Q3 = Q2 * Q, P3 = P * P * P;
    constexpr int SX = 1, SY = L::PITCH, SZ = L::PLANE;
    constexpr int NOH = (Q + 1) / 2;
    static_assert(G * Q2 <= NT, "one line per lane");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *const A = reinterpret_cast<T *>(smem_raw);
    T *const Bb = MODE == kMass ? A : A + G * L::ELEM;
    T *const C = MODE == kMass ? A : Bb + G * L::ELEM;
    double *const sC = reinterpret_cast<double *>(A + line_array_len<P, Q, T>(MODE, G));
    const int tid = threadIdx.x;
    const LinePos pos = line_pos_of<G>(a, blockIdx.x, gridDim.x);
    const int vec = blockIdx.y;
    const cptr<T> bas = (cptr<T>)(uintptr_t)a.bas;
    const int nx = a.nex * p + 1, ny = a.ney * p + 1, nz = a.nez * p + 1;

    // Lane roles, packed into three registers for the whole march (an inactive role has its bit clear):
    //   X line (row b, plane k) and Z line (a, b): LDS positions; Y line: node column X, plane k
    static_assert(G * L::ELEM < 1 << 14, "positions in 14 bits");
    constexpr uint32_t kAct = 1u << 14, kDual = 1u << 15;
    uint32_t rxz, ry, rz;
    int X, ky;
    {
        ky = tid / W;
        X = tid - ky * W;
        int g = 0, i = X;
        if constexpr (G > 1) {
            g = X / p;
            if (g > pos.nvalid - 1) g = pos.nvalid - 1;
            i = X - g * p;
        }
        ry = 0;
        if (tid < W * P && X <= pos.nvalid * p)
            ry = (uint32_t)(g * L::ELEM + ky * SZ + i) | kAct | (G > 1 && i == 0 && g > 0 ? kDual : 0u);  // dual: face shared with g-1
        const int bx = tid % Q, kx = (tid / Q) % P, gx = tid / (Q * P);
        rxz = 0;
        if (tid < G * P * Q && gx < pos.nvalid) rxz = (uint32_t)(gx * L::ELEM + kx * SZ + bx * SY) | kAct;
        const int az = tid % Q, bz = (tid / Q) % Q, gz = tid / Q2;
        if (tid < G * Q2 && gz < pos.nvalid) rxz |= ((uint32_t)(gz * L::ELEM + bz * SY + az) | kAct) << 16;
        rz = (uint32_t)az | (uint32_t)bz << 4 | (uint32_t)gz << 8;
    }
    const auto at = [](uint32_t r) { return (int)(r & (kAct - 1)); };
    // the group's first node is uniform; a lane adds its own offset (OFF: 32 bits where a slab of P planes allows)
    const int64_t stride = (int64_t)nx * a.nvec;
    const int64_t node0 = (((int64_t)pos.ez * p * ny + (int64_t)pos.ey0 * p) * nx + (int64_t)pos.ex0 * p) * a.nvec + vec;
    const T *xb = a.x + node0;
    T *yb = DET ? nullptr : a.y + node0;
    const int I = pos.ex0 * p + X, K = pos.ez * p + ky;
    const bool io = (ry & kAct) && !(a.dirichlet && (I == 0 || I == nx - 1 || K == 0 || K == nz - 1));
    const OFF lane0 = ((OFF)ky * (OFF)ny * (OFF)nx + (OFF)X) * (OFF)a.nvec;

    T xv[P], carry = T(0);
#pragma unroll
    for (int j = 0; j < P; ++j) xv[j] = io ? (xb + j * stride)[lane0] : T(0);

    // Vertices: two y-planes of 2 (G + 1) vertices in LDS, used in turn; a march loads one plane per element.  The
    // elements' trilinear coefficients are formed from them in the X stage.
    constexpr int VP = 6 * (G + 1), RV = (VP + NT - 1) / NT, RC = (G * kTriCoef + NT - 1) / NT;
    double *const sV = sC + G * kTriCoef + 2 * Q;
    double vtx[RV];
    auto vtx_load = [&](int vy) {
#pragma unroll
        for (int r = 0; r < RV; ++r) {
            const int t = tid + r * NT, z = t / (VP / 2), c = t - z * (VP / 2);
            if (t < VP && c < 3 * (pos.nvalid + 1))
                vtx[r] = a.vert[3 * (pos.ex0 + (int64_t)(a.nex + 1) * (vy + (int64_t)(a.ney + 1) * (pos.ez + z))) + c];
        }
    };
    auto vtx_store = [&](int vy) {
#pragma unroll
        for (int r = 0; r < RV; ++r)
            if (tid + r * NT < VP) sV[(vy & 1) * VP + tid + r * NT] = vtx[r];
    };
    vtx_load(pos.ey0);
    vtx_store(pos.ey0);
    vtx_load(pos.ey0 + 1);
    // points, then weights (contiguous in the basis block)
    double *const sR = sC + G * kTriCoef;
    if (tid < 2 * Q) sR[tid] = a.bas64[basis_xq(P, Q) + tid];
    for (int ey = pos.ey0; ey < pos.ey1; ++ey) {
        const bool more = ey + 1 < pos.ey1;
        cptr<T> Bf, Gf;
        auto matrices = [&]() {
            const cptr<T> b = opaque<T>(bas);
            Bf = b + basis_bf(P, Q);
            Gf = b + (COLLOC ? basis_df(P, Q) : basis_gf(P, Q));
        };
        matrices();
        // --- Y -----------------------------------------------------------------------------
        vtx_store(ey + 1);
        if (ry & kAct) {
            const int ly = at(ry), ly2 = ly - L::ELEM + p;
            T v[P];
#pragma unroll
            for (int j = 0; j < P; ++j) v[j] = xv[j];
            if (a.dirichlet) {
                if (ey == 0) v[0] = T(0);
                if (ey == a.ney - 1) v[P - 1] = T(0);
            }
            Folded<P, T> f;
            f.set(v);
            auto put = [&](T *arr, int o, T lo, T hi) {
                arr[ly + o * SY] = lo;
                if (2 * o + 1 != Q) arr[ly + (Q - 1 - o) * SY] = hi;
                if (ry & kDual) {
                    arr[ly2 + o * SY] = lo;
                    if (2 * o + 1 != Q) arr[ly2 + (Q - 1 - o) * SY] = hi;
                }
            };
            if constexpr (COLLOC) {
#pragma unroll
                for (int o = 0; o < NOH; ++o) put(A, o, v[o], v[P - 1 - o]);
            } else {
                line_all<P, Q, 1>(Bf, f, [&](int o, T lo, T hi) { put(A, o, lo, hi); });
            }
            if constexpr (MODE == kDiff) line_all<P, Q, -1>(Gf, f, [&](int o, T lo, T hi) { put(Bb, o, lo, hi); });
        }
        group_sync<NT>();
        // --- X -----------------------------------------------------------------------------
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            int t = tid + r * NT;
            asm volatile("" : "+v"(t));  // (addresses not kept through the other stages)
            if (t < pos.nvalid * kTriCoef) {
                const int g = t / kTriCoef, c = t - g * kTriCoef, m = c / 3;
                sC[t] = tri_coef(sV + 3 * g + (c - 3 * m), (ey & 1) * VP, VP - (ey & 1) * VP, VP / 2, m + 1);
            }
        }
        if (rxz & kAct) {
            const int lx = at(rxz);
            matrices();
            T v[P];
            Folded<P, T> f;
            auto put = [&](T *arr, int o, T lo, T hi) {
                arr[lx + o * SX] = lo;
                if (2 * o + 1 != Q) arr[lx + (Q - 1 - o) * SX] = hi;
            };
            line_read<P, SX>(A + lx, v);
            f.set(v);
            if constexpr (MODE == kDiff) line_all<P, Q, -1>(Gf, f, [&](int o, T lo, T hi) { put(C, o, lo, hi); });
            if constexpr (!COLLOC) {
                line_all<P, Q, 1>(Bf, f, [&](int o, T lo, T hi) { put(A, o, lo, hi); });
                if constexpr (MODE == kDiff) {
                    line_read<P, SX>(Bb + lx, v);
                    f.set(v);
                    line_all<P, Q, 1>(Bf, f, [&](int o, T lo, T hi) { put(Bb, o, lo, hi); });
                }
            }
        }
        group_sync<NT>();
        // --- Z -----------------------------------------------------------------------------
        if (rxz >> 16 & kAct) {
            const int lz = at(rxz >> 16), az = rz & 15, bz = rz >> 4 & 15, gz = rz >> 8;
            const cptr<double> xq = (cptr<double>)(uintptr_t)a.bas64 + basis_xq(P, Q);
            const cptr<double> wq = (cptr<double>)(uintptr_t)a.bas64 + basis_wq(P, Q);
            matrices();
            T v[P];
            Folded<P, T> f;
            T ur[Q], us[Q], ut[Q];
            auto pair_to = [&](T (&u)[Q], int o, T lo, T hi) {
                u[o] = lo;
                if (2 * o + 1 != Q) u[Q - 1 - o] = hi;
            };
            line_read<P, SZ>(A + lz, v);
            f.set(v);
            if constexpr (MODE == kMass) {
                line_all<P, Q, 1>(Bf, f, [&](int o, T lo, T hi) { pair_to(ut, o, lo, hi); });
                ZLineGeom g;
                g.set(sC + gz * kTriCoef, sR[az], sR[bz]);
                const double wz = sR[Q + az] * sR[Q + bz];
                double d[3];
                g.det_poly(d);
#pragma unroll
                for (int c = 0; c < Q; ++c) ut[c] *= T((wz * wq[c]) * (d[0] + xq[c] * (d[1] + xq[c] * d[2])));
                TransAcc<P, T> t;
                t.zero();
                t.template add<Q, 1>(Bf, ut);
#pragma unroll
                for (int k = 0; k < P; ++k) A[lz + k * SZ] = t.out(k);
            } else {
                line_all<P, Q, -1>(Gf, f, [&](int o, T lo, T hi) { pair_to(ut, o, lo, hi); });
                if constexpr (COLLOC) {
                    line_read<Q, SZ>(Bb + lz, us);
                    line_read<Q, SZ>(C + lz, ur);
                } else {
                    line_read<P, SZ>(Bb + lz, v);
                    f.set(v);
                    line_all<P, Q, 1>(Bf, f, [&](int o, T lo, T hi) { pair_to(us, o, lo, hi); });
                    line_read<P, SZ>(C + lz, v);
                    f.set(v);
                    line_all<P, Q, 1>(Bf, f, [&](int o, T lo, T hi) { pair_to(ur, o, lo, hi); });
                }
                const double *kp = nullptr;
                if constexpr (VARK)
                    kp = a.kappa + (pos.ex0 + gz + (int64_t)a.nex * (ey + (int64_t)a.ney * pos.ez)) * Q3 + bz * Q + az;
                ZLineGeom g;
                g.set(sC + gz * kTriCoef, sR[az], sR[bz]);
                const double wz = sR[Q + az] * sR[Q + bz];
#pragma unroll
                for (int c = 0; c < Q; ++c) {
                    // one point at a time: evaluated together the points' temporaries would spill
                    g.pin();
                    double w = wz * wq[c];
                    if constexpr (VARK) w *= kp[c * Q2];
                    double r = ur[c], s = us[c], t = ut[c];
                    apply_geom(g, xq[c], w, r, s, t);
                    ur[c] = T(r);
                    us[c] = T(s);
                    ut[c] = T(t);
                    asm volatile("" : "+v"(ur[c]), "+v"(us[c]), "+v"(ut[c]));
                }
                __builtin_amdgcn_sched_barrier(0);
                matrices();
                TransAcc<P, T> t;
                t.zero();
                t.template add<Q, -1>(Gf, ut);
#pragma unroll
                for (int k = 0; k < P; ++k) A[lz + k * SZ] = t.out(k);
                if constexpr (COLLOC) {
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        Bb[lz + k * SZ] = us[k];
                        C[lz + k * SZ] = ur[k];
                    }
                } else {
                    t.zero();
                    t.template add<Q, 1>(Bf, us);
#pragma unroll
                    for (int k = 0; k < P; ++k) Bb[lz + k * SZ] = t.out(k);
                    t.zero();
                    t.template add<Q, 1>(Bf, ur);
#pragma unroll
                    for (int k = 0; k < P; ++k) C[lz + k * SZ] = t.out(k);
                }
            }
        }
        // the next element's inputs travel behind the transposed stages
        if (more) {
            xv[0] = xv[P - 1];
            xb += p * stride;
            if (io) {
                gptr<const T> row = (gptr<const T>)xb;
#pragma unroll
                for (int j = 1; j < P; ++j) {
                    row += stride;
                    asm volatile("" : "+s"(row));
                    xv[j] = row[lane0];
                }
            }
            vtx_load(ey + 2);
        }
        group_sync<NT>();
        // --- X^T ---------------------------------------------------------------------------
        if (rxz & kAct) {
            const int lx = at(rxz);
            matrices();
            T w[Q];
            TransAcc<P, T> t;
            t.zero();
            if constexpr (COLLOC) {
                line_read<Q, SX>(C + lx, w);
                t.template add<Q, -1>(Gf, w);
#pragma unroll
                for (int i = 0; i < P; ++i) A[lx + i] += t.out(i);
            } else {
                line_read<Q, SX>(A + lx, w);
                t.template add<Q, 1>(Bf, w);
                if constexpr (MODE == kDiff) {
                    line_read<Q, SX>(C + lx, w);
                    t.template add<Q, -1>(Gf, w);
                }
#pragma unroll
                for (int i = 0; i < P; ++i) A[lx + i] = t.out(i);
                if constexpr (MODE == kDiff) {
                    line_read<Q, SX>(Bb + lx, w);
                    t.zero();
                    t.template add<Q, 1>(Bf, w);
#pragma unroll
                    for (int i = 0; i < P; ++i) Bb[lx + i] = t.out(i);
                }
            }
        }
        group_sync<NT>();
        // --- Y^T and scatter ---------------------------------------------------------------
        auto transposed_y = [&](int base, bool two, int base2, T (&out)[P]) {
            // a column shared by two elements of the group: both elements' lines summed first (the
            // contraction is linear)
            matrices();
            T w[Q];
            TransAcc<P, T> t;
            t.zero();
            auto get = [&](const T *arr) {
                line_read<Q, SY>(arr + base, w);
                if (two) {
#pragma unroll
                    for (int b = 0; b < Q; ++b) w[b] += arr[base2 + b * SY];
                }
            };
            if constexpr (COLLOC) {
                get(Bb);
                t.template add<Q, -1>(Gf, w);
                get(A);
#pragma unroll
                for (int j = 0; j < P; ++j) out[j] = t.out(j) + w[j];
            } else {
                get(A);
                t.template add<Q, 1>(Bf, w);
                if constexpr (MODE == kDiff) {
                    get(Bb);
                    t.template add<Q, -1>(Gf, w);
                }
#pragma unroll
                for (int j = 0; j < P; ++j) out[j] = t.out(j);
            }
        };
        if constexpr (DET) {
            // element values as they are: one line per element column
            const int i = tid % P, k = (tid / P) % P, g = tid / (P * P);
            if (tid < G * P * P && g < pos.nvalid) {
                T out[P];
                transposed_y(g * L::ELEM + k * SZ + i, false, 0, out);
                const int64_t e = pos.ex0 + g + (int64_t)a.nex * (ey + (int64_t)a.ney * pos.ez);
                T *eb = a.ebuf + (e * P3 + i + P * P * k) * a.nvec + vec;
#pragma unroll
                for (int j = 0; j < P; ++j) eb[j * P * a.nvec] = out[j];
            }
        } else if (io) {
            T out[P];
            transposed_y(at(ry), ry & kDual, at(ry) - L::ELEM + p, out);
            out[0] += carry;
            carry = out[P - 1];
            const bool m0 = a.dirichlet && ey == 0, m1 = a.dirichlet && ey == a.ney - 1;
            // one row address at a time in scalar registers
            gptr<T> row = (gptr<T>)yb;
            if (!m0) global_add(row + lane0, out[0]);
#pragma unroll
            for (int j = 1; j < P - 1; ++j) {
                row += stride;
                asm volatile("" : "+s"(row) : "v"(out[j]));
                global_add(row + lane0, out[j]);
            }
            if (!more && !m1) global_add(row + stride + lane0, out[P - 1]);
        }
        yb += p * stride;
        if (more) group_sync<NT>();
    }
}

// ---------------------------------------------------------------------------
// Collocated diffusion, VC vectors of a multi-vector together: the stages of
// k_line with the vector as the fastest lane index, so that a gather, an LDS
// access and an atomic touch runs of VC consecutive values (64 bytes for 8
// FP64 vectors).  The factors are the stored ones: lane v of the VC lanes of a
// z-line loads the six factors of the points v, v + VC, ... one element ahead,
// and the others take them by DPP broadcasts inside the group, 12 moves a point
// in place of six loads.  (Factors evaluated in the kernel as in k_line read
// half the bytes but took 267 against 254 us at p = 6, 294 against 272 at p = 5
// and 411 against 344 at p = 2, 3e6 nodes of 8 vectors; they won at p = 7 and 8
// only, 354 against 370 and 395 against 442.)
// Measured, k_apply with chunks before and this now, FP64: p = 6, 8 vectors of
// 1e7 nodes 1766 -> 868 us (1.6 GB of 8-vector data), p = 3, 12 vectors of 1e6
// nodes 280 -> 193.  The LDS of two groups of 7 wavefronts fills a CU at p = 6:
// 883 us become 694 without the atomics, 577 without the loads as well, and 521
// without barriers, so that memory and the stages' latency share the time; the
// vector units are busy for 35% of it.
// ---------------------------------------------------------------------------

// The value of lane K of each group of VC lanes (VC = 4: a quad; 8: half a row of 16).
template <int VC, int K>
__device__ __forceinline__ double lane_bcast(double v)
{
    static_assert(VC == 4 || VC == 8, "groups of 4 or 8 lanes");
    if constexpr (VC == 8) {
        const long s = __builtin_bit_cast(long, v);
        const long lo = __builtin_amdgcn_update_dpp(s, s, 0x150 + K, 0xf, 0xf, false);      // row_newbcast
        const long hi = __builtin_amdgcn_update_dpp(lo, s, 0x150 + K + 8, 0xf, 0xc, false);  // upper half of the row
        return __builtin_bit_cast(double, hi);
    } else {
        const int2 s = __builtin_bit_cast(int2, v);
        int2 r;  // quad_perm
        r.x = __builtin_amdgcn_update_dpp(s.x, s.x, K * 0x55, 0xf, 0xf, false);
        r.y = __builtin_amdgcn_update_dpp(s.y, s.y, K * 0x55, 0xf, 0xf, false);
        return __builtin_bit_cast(double, r);
    }
}
template <int VC, int K>
__device__ __forceinline__ float lane_bcast(float v)
{
    const int s = __builtin_bit_cast(int, v);
    if constexpr (VC == 8) {
        const int lo = __builtin_amdgcn_update_dpp(s, s, 0x150 + K, 0xf, 0xf, false);
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(lo, s, 0x150 + K + 8, 0xf, 0xc, false));
    } else {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(s, s, K * 0x55, 0xf, 0xf, false));
    }
}

template <typename F, int... I>
__device__ __forceinline__ void static_for_seq(F f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F f)
{
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

template <int Q, int VC, typename T>
constexpr size_t mline_lds(int G)
{
    return (size_t)3 * G * LineLds<Q, Q>::ELEM * VC * sizeof(T);
}

template <int Q, int VC, typename T, int G, int NT, typename OFF>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
k_mline(const LineArgs<T> a)
{
    using L = LineLds<Q, Q>;
    constexpr int P = Q, p = P - 1, W = G * p + 1, Q2 = Q * Q;
    constexpr int SX = VC, SY = L::PITCH * VC, SZ = L::PLANE * VC, ELEM = L::ELEM * VC;
    constexpr int NM = (Q + VC - 1) / VC;  // points of a z-line whose factors one lane computes
    static_assert(G * Q2 * VC <= NT, "one line per lane");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *const A = reinterpret_cast<T *>(smem_raw), *const Bb = A + G * ELEM, *const C = Bb + G * ELEM;
    const int tid = threadIdx.x, vc = tid % VC, lt = tid / VC;
    // chunks of vectors fastest: those of one element run side by side and share its lines in the L2
    const unsigned nch = (a.nvec + VC - 1) / VC;
    const unsigned xcd = blockIdx.x % kNumXcd, nq = gridDim.x / kNumXcd, nr = gridDim.x % kNumXcd;
    const unsigned bid = a.base + xcd * nq + (xcd < nr ? xcd : nr) + blockIdx.x / kNumXcd;
    const int vec = (int)(bid % nch) * VC + vc;
    LinePos pos;
    {
        const unsigned g = bid / nch, r = g / (unsigned)a.ngx;
        pos.ex0 = (int)(g % (unsigned)a.ngx) * G;
        pos.nvalid = a.nex - pos.ex0 < G ? a.nex - pos.ex0 : G;
        pos.ey0 = (int)(r % (unsigned)a.nych) * a.march;
        pos.ey1 = pos.ey0 + a.march < a.ney ? pos.ey0 + a.march : a.ney;
        pos.ez = (int)(r / (unsigned)a.nych);
    }
    const cptr<T> bas = (cptr<T>)(uintptr_t)a.bas;
    const int nx = a.nex * p + 1, ny = a.ney * p + 1, nz = a.nez * p + 1;

    // lane roles as in k_line, of line lt and vector vc
    static_assert(G * ELEM < 1 << 14, "positions in 14 bits");
    constexpr uint32_t kAct = 1u << 14, kDual = 1u << 15;
    uint32_t rxz, ry, rz;
    const int ky = lt / W, X = lt - ky * W;
    {
        int g = 0, i = X;
        if constexpr (G > 1) {
            g = X / p;
            if (g > pos.nvalid - 1) g = pos.nvalid - 1;
            i = X - g * p;
        }
        ry = 0;
        if (lt < W * P && X <= pos.nvalid * p)
            ry = (uint32_t)(g * ELEM + ky * SZ + i * SX + vc) | kAct | (G > 1 && i == 0 && g > 0 ? kDual : 0u);
        const int bx = lt % Q, kx = (lt / Q) % Q, gx = lt / Q2;
        rxz = 0;
        if (lt < G * Q2 && gx < pos.nvalid)  // row b of plane k, and z-line (a, b)
            rxz = (uint32_t)(gx * ELEM + kx * SZ + bx * SY + vc) | kAct |
                  ((uint32_t)(gx * ELEM + kx * SY + bx * SX + vc) | kAct) << 16;
        rz = (uint32_t)bx | (uint32_t)kx << 4 | (uint32_t)gx << 8;
    }
    const auto at = [](uint32_t r) { return (int)(r & (kAct - 1)); };
    const int64_t stride = (int64_t)nx * a.nvec;
    const int64_t node0 = (((int64_t)pos.ez * p * ny + (int64_t)pos.ey0 * p) * nx + (int64_t)pos.ex0 * p) * a.nvec;
    const T *xb = a.x + node0;
    T *yb = a.y + node0;
    const int I = pos.ex0 * p + X, K = pos.ez * p + ky;
    const bool io = (ry & kAct) && vec < a.nvec && !(a.dirichlet && (I == 0 || I == nx - 1 || K == 0 || K == nz - 1));
    const OFF lane0 = ((OFF)ky * (OFF)ny * (OFF)nx + (OFF)X) * (OFF)a.nvec + (OFF)vec;

    T xv[P], carry = T(0);
#pragma unroll
    for (int j = 0; j < P; ++j) xv[j] = io ? (xb + j * stride)[lane0] : T(0);
    // factors of this lane's points (a, b, vc + m VC) of the element at ey
    T gm[NM][kQdDiff];
    auto q_load = [&](int ey) {
        if (rxz >> 16 & kAct) {
            const int64_t e = pos.ex0 + (int)(rz >> 8) + (int64_t)a.nex * (ey + (int64_t)a.ney * pos.ez);
            const T *qd = a.qdata + e * (kQdDiff * Q2 * Q) + (rz >> 4 & 15) * Q + (rz & 15);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int c = vc + m * VC < Q ? vc + m * VC : Q - 1;
#pragma unroll
                for (int i = 0; i < kQdDiff; ++i) gm[m][i] = __builtin_nontemporal_load(&qd[i * Q2 * Q + c * Q2]);
            }
        }
    };
    q_load(pos.ey0);

    for (int ey = pos.ey0; ey < pos.ey1; ++ey) {
        const bool more = ey + 1 < pos.ey1;
        cptr<T> Df;
        auto matrices = [&]() { Df = opaque<T>(bas) + basis_df(P, Q); };
        matrices();
        // --- Y -----------------------------------------------------------------------------
        if (ry & kAct) {
            const int ly = at(ry), ly2 = ly - ELEM + p * SX;
            T v[P];
#pragma unroll
            for (int j = 0; j < P; ++j) v[j] = xv[j];
            if (a.dirichlet) {
                if (ey == 0) v[0] = T(0);
                if (ey == a.ney - 1) v[P - 1] = T(0);
            }
            Folded<P, T> f;
            f.set(v);
            auto put = [&](T *arr, int o, T lo, T hi) {
                arr[ly + o * SY] = lo;
                if (2 * o + 1 != Q) arr[ly + (Q - 1 - o) * SY] = hi;
                if (ry & kDual) {
                    arr[ly2 + o * SY] = lo;
                    if (2 * o + 1 != Q) arr[ly2 + (Q - 1 - o) * SY] = hi;
                }
            };
#pragma unroll
            for (int o = 0; o < (Q + 1) / 2; ++o) put(A, o, v[o], v[P - 1 - o]);
            line_all<P, Q, -1>(Df, f, [&](int o, T lo, T hi) { put(Bb, o, lo, hi); });
        }
        // the next element's inputs travel behind all the stages that follow
        if (more) {
            xv[0] = xv[P - 1];
            xb += p * stride;
            if (io) {
                gptr<const T> row = (gptr<const T>)xb;
#pragma unroll
                for (int j = 1; j < P; ++j) {
                    row += stride;
                    asm volatile("" : "+s"(row));
                    xv[j] = row[lane0];
                }
            }
        }
        group_sync<NT>();
        // --- X -----------------------------------------------------------------------------
        if (rxz & kAct) {
            const int lx = at(rxz);
            matrices();
            T v[P];
            Folded<P, T> f;
            line_read<P, SX>(A + lx, v);
            f.set(v);
            line_all<P, Q, -1>(Df, f, [&](int o, T lo, T hi) {
                C[lx + o * SX] = lo;
                if (2 * o + 1 != Q) C[lx + (Q - 1 - o) * SX] = hi;
            });
        }
        group_sync<NT>();
        // --- Z -----------------------------------------------------------------------------
        if (rxz >> 16 & kAct) {
            const int lz = at(rxz >> 16);
            matrices();
            T v[P], ur[Q], us[Q], ut[Q];
            Folded<P, T> f;
            line_read<P, SZ>(A + lz, v);
            f.set(v);
            line_all<P, Q, -1>(Df, f, [&](int o, T lo, T hi) {
                ut[o] = lo;
                if (2 * o + 1 != Q) ut[Q - 1 - o] = hi;
            });
            line_read<Q, SZ>(Bb + lz, us);
            line_read<Q, SZ>(C + lz, ur);
            static_for<Q>([&](auto ci) {
                constexpr int c = ci, m = c / VC, k = c % VC;
                T g[kQdDiff];
#pragma unroll
                for (int i = 0; i < kQdDiff; ++i) g[i] = lane_bcast<VC, k>(gm[m][i]);
                const T r = ur[c], s = us[c], t = ut[c];
                ur[c] = g[0] * r + g[5] * s + g[4] * t;
                us[c] = g[5] * r + g[1] * s + g[3] * t;
                ut[c] = g[4] * r + g[3] * s + g[2] * t;
                asm volatile("" : "+v"(ur[c]), "+v"(us[c]), "+v"(ut[c]));  // one point's factors at a time
            });
            matrices();
            TransAcc<P, T> t;
            t.zero();
            t.template add<Q, -1>(Df, ut);
#pragma unroll
            for (int k = 0; k < P; ++k) {
                A[lz + k * SZ] = t.out(k);
                Bb[lz + k * SZ] = us[k];
                C[lz + k * SZ] = ur[k];
            }
        }
        if (more) q_load(ey + 1);
        group_sync<NT>();
        // --- X^T ---------------------------------------------------------------------------
        if (rxz & kAct) {
            const int lx = at(rxz);
            matrices();
            T w[Q];
            TransAcc<P, T> t;
            t.zero();
            line_read<Q, SX>(C + lx, w);
            t.template add<Q, -1>(Df, w);
#pragma unroll
            for (int i = 0; i < P; ++i) A[lx + i * SX] += t.out(i);
        }
        group_sync<NT>();
        // --- Y^T and scatter ---------------------------------------------------------------
        if (io) {
            const int ly = at(ry), ly2 = ly - ELEM + p * SX;
            matrices();
            T w[Q], out[P];
            TransAcc<P, T> t;
            t.zero();
            auto get = [&](const T *arr) {
                line_read<Q, SY>(arr + ly, w);
                if (ry & kDual) {
#pragma unroll
                    for (int b = 0; b < Q; ++b) w[b] += arr[ly2 + b * SY];
                }
            };
            get(Bb);
            t.template add<Q, -1>(Df, w);
            get(A);
#pragma unroll
            for (int j = 0; j < P; ++j) out[j] = t.out(j) + w[j];
            out[0] += carry;
            carry = out[P - 1];
            const bool m0 = a.dirichlet && ey == 0, m1 = a.dirichlet && ey == a.ney - 1;
            gptr<T> row = (gptr<T>)yb;
            if (!m0) global_add(row + lane0, out[0]);
#pragma unroll
            for (int j = 1; j < P - 1; ++j) {
                row += stride;
                asm volatile("" : "+s"(row) : "v"(out[j]));
                global_add(row + lane0, out[j]);
            }
            if (!more && !m1) global_add(row + stride + lane0, out[P - 1]);
        }
        yb += p * stride;
        if (more) group_sync<NT>();
    }
}

// ---------------------------------------------------------------------------
// Coefficient gradient g[e][pt] = (Dhat r)^T G0 (Dhat u) at every point: the
// forward stages of k_line for both vectors at once, on neighbouring lanes (u
// even, r odd).  The lanes of a pair share the points of their z-line, o of the
// one and Q-1-o of the other, the two outputs that a folded row gives: a lane
// forms E +- O and E -+ O with the signs of its side, keeps its own point's
// value and hands the other one over by a DPP swap, so that the geometry of a
// point is evaluated once (both lanes at every point: 238 against 219 us at
// p = 6, 327 against 314 at p = 4, 1e7 nodes).
// Before, one element per wavefront with six LDS arrays and stored factors, and
// now: Gauss, 1e7 nodes, p = 4 510 -> 314 us, p = 6 434 -> 219; 3e6 nodes,
// p = 2 370 -> 191, p = 8 154 -> 69.  p = 4 moves 0.56 GB (107 us); the vector
// units are busy 56% of the time, the rest is the latency of three stages.
// ---------------------------------------------------------------------------
struct KgradArgs {
    const double *bas, *vert, *u, *r;
    double *g;
    int nex, ney, nez, dirichlet;
    int ngx, nych, march;
    unsigned base;
};

// The value of the other lane of the pair.
__device__ __forceinline__ double lane_swap(double v)
{
    int2 s = __builtin_bit_cast(int2, v);
    s.x = __builtin_amdgcn_update_dpp(s.x, s.x, 0xb1, 0xf, 0xf, false);  // quad_perm [1, 0, 3, 2]
    s.y = __builtin_amdgcn_update_dpp(s.y, s.y, 0xb1, 0xf, 0xf, false);
    return __builtin_bit_cast(double, s);
}

template <int P, int Q>
constexpr size_t kgrad_lds(int G)
{
    return ((size_t)6 * G * LineLds<P, Q>::ELEM + (size_t)G * kTriCoef + 2 * Q + 12 * (G + 1)) * 8;
}

// STACK: the G elements of a group are consecutive in z instead of x, for rows that leave part of a group idle; the face
// between two of them is then loaded twice.  At 2e6 nodes, groups in x and stacked: Gauss p = 1, rows of 1, 2, 4, 9 950 210,
// 706 317, 541 386, 584 430 us; p = 3, rows of 1, 3, 6 138 55, 80 66, 96 69; collocated p = 2, rows of 1, 8 155 44, 86 64; a
// cube of 3e6 nodes, 0.97 to 1.05 of the time.
template <int P, int Q, bool COLLOC, int G, int NT, bool STACK>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(line_waves(Q, kDiff))))
k_kgrad(const KgradArgs a)
{
    using L = LineLds<P, Q>;
    using T = double;
    constexpr int p = P - 1, W = STACK ? P : G * p + 1, Q2 = Q * Q, Q3 = Q2 * Q;
    constexpr int SX = 2, SY = L::PITCH * 2, SZ = L::PLANE * 2, ELEM = L::ELEM * 2;
    constexpr int NOH = (Q + 1) / 2;
    static_assert(2 * G * Q2 <= NT, "one line of one vector per lane");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *const A = reinterpret_cast<T *>(smem_raw), *const Bb = A + G * ELEM, *const C = Bb + G * ELEM;
    T *const sC = C + G * ELEM;
    const int tid = threadIdx.x, vec = tid & 1, lt = tid >> 1;
    LinePos pos = line_pos_of<STACK ? 1 : G>(a, blockIdx.x, gridDim.x);
    if constexpr (STACK) {
        pos.ez *= G;
        pos.nvalid = a.nez - pos.ez < G ? a.nez - pos.ez : G;
    }
    const cptr<T> bas = (cptr<T>)(uintptr_t)a.bas;
    const int nx = a.nex * p + 1, ny = a.ney * p + 1, nz = a.nez * p + 1;

    // lane roles as in k_line, of line lt and vector vec
    static_assert(G * ELEM < 1 << 14, "positions in 14 bits");
    constexpr uint32_t kAct = 1u << 14, kDual = 1u << 15;
    uint32_t rxz, ry, rz;
    int ky = lt / W, X = lt - ky * W, gy = 0;  // (stacked: plane ky of element gy)
    if constexpr (STACK) gy = ky / P, ky -= gy * P;
    {
        int g = gy, i = X;
        if constexpr (G > 1 && !STACK) {
            g = X / p;
            if (g > pos.nvalid - 1) g = pos.nvalid - 1;
            i = X - g * p;
        }
        ry = 0;
        if (STACK ? gy < pos.nvalid : lt < W * P && X <= pos.nvalid * p)
            ry = (uint32_t)(g * ELEM + ky * SZ + i * SX + vec) | kAct |
                 (G > 1 && !STACK && i == 0 && g > 0 ? kDual : 0u);
        const int bx = lt % Q, kx = (lt / Q) % P, gx = lt / (Q * P);
        rxz = 0;
        if (lt < G * P * Q && gx < pos.nvalid) rxz = (uint32_t)(gx * ELEM + kx * SZ + bx * SY + vec) | kAct;
        const int az = lt % Q, bz = (lt / Q) % Q, gz = lt / Q2;
        if (lt < G * Q2 && gz < pos.nvalid) rxz |= ((uint32_t)(gz * ELEM + bz * SY + az * SX + vec) | kAct) << 16;
        rz = (uint32_t)az | (uint32_t)bz << 4 | (uint32_t)gz << 8;
    }
    const auto at = [](uint32_t v) { return (int)(v & (kAct - 1)); };
    const int I = pos.ex0 * p + X, K = (pos.ez + gy) * p + ky;
    const bool io = (ry & kAct) && !(a.dirichlet && (I == 0 || I == nx - 1 || K == 0 || K == nz - 1));
    gptr<const T> xb = (gptr<const T>)(vec ? a.r : a.u) + ((int64_t)K * ny + (int64_t)pos.ey0 * p) * nx + I;

    T xv[P];
#pragma unroll
    for (int j = 0; j < P; ++j) xv[j] = io ? xb[(int64_t)j * nx] : T(0);

    // vertices and trilinear coefficients as in k_line (stacked: G + 1 planes of 2 x 2 vertices in use, two per y-plane)
    constexpr int VZ = STACK ? 6 : 3 * (G + 1);  // values of one z-plane of a y-plane
    constexpr int VP = 6 * (G + 1), RV = (VP + NT - 1) / NT, RC = (G * kTriCoef + NT - 1) / NT;
    T *const sR = sC + G * kTriCoef, *const sV = sR + 2 * Q;
    double vtx[RV];
    auto vtx_load = [&](int vy) {
#pragma unroll
        for (int r = 0; r < RV; ++r) {
            const int t = tid + r * NT, z = t / VZ, c = t - z * VZ;
            if (t < VP && (STACK ? z <= pos.nvalid : c < 3 * (pos.nvalid + 1)))
                vtx[r] = a.vert[3 * (pos.ex0 + (int64_t)(a.nex + 1) * (vy + (int64_t)(a.ney + 1) * (pos.ez + z))) + c];
        }
    };
    auto vtx_store = [&](int vy) {
#pragma unroll
        for (int r = 0; r < RV; ++r)
            if (tid + r * NT < VP) sV[(vy & 1) * VP + tid + r * NT] = vtx[r];
    };
    vtx_load(pos.ey0);
    vtx_store(pos.ey0);
    vtx_load(pos.ey0 + 1);
    if (tid < 2 * Q) sR[tid] = a.bas[basis_xq(P, Q) + tid];
    for (int ey = pos.ey0; ey < pos.ey1; ++ey) {
        const bool more = ey + 1 < pos.ey1;
        cptr<T> Bf, Gf;
        auto matrices = [&]() {
            const cptr<T> b = opaque<T>(bas);
            Bf = b + basis_bf(P, Q);
            Gf = b + (COLLOC ? basis_df(P, Q) : basis_gf(P, Q));
        };
        matrices();
        // --- Y -----------------------------------------------------------------------------
        vtx_store(ey + 1);
        if (ry & kAct) {
            const int ly = at(ry), ly2 = ly - ELEM + p * SX;
            T v[P];
#pragma unroll
            for (int j = 0; j < P; ++j) v[j] = xv[j];
            if (a.dirichlet) {
                if (ey == 0) v[0] = T(0);
                if (ey == a.ney - 1) v[P - 1] = T(0);
            }
            Folded<P, T> f;
            f.set(v);
            auto put = [&](T *arr, int o, T lo, T hi) {
                arr[ly + o * SY] = lo;
                if (2 * o + 1 != Q) arr[ly + (Q - 1 - o) * SY] = hi;
                if (ry & kDual) {
                    arr[ly2 + o * SY] = lo;
                    if (2 * o + 1 != Q) arr[ly2 + (Q - 1 - o) * SY] = hi;
                }
            };
            if constexpr (COLLOC) {
#pragma unroll
                for (int o = 0; o < NOH; ++o) put(A, o, v[o], v[P - 1 - o]);
            } else {
                line_all<P, Q, 1>(Bf, f, [&](int o, T lo, T hi) { put(A, o, lo, hi); });
            }
            line_all<P, Q, -1>(Gf, f, [&](int o, T lo, T hi) { put(Bb, o, lo, hi); });
        }
        if (more) {
            vtx_load(ey + 2);
            xv[0] = xv[P - 1];
            xb += (int64_t)p * nx;
            if (io) {
#pragma unroll
                for (int j = 1; j < P; ++j) xv[j] = xb[(int64_t)j * nx];
            }
        }
        group_sync<NT>();
        // --- X -----------------------------------------------------------------------------
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            int t = tid + r * NT;
            asm volatile("" : "+v"(t));
            if (t < pos.nvalid * kTriCoef) {
                const int g = t / kTriCoef, c = t - g * kTriCoef, m = c / 3;
                sC[t] = tri_coef(sV + (STACK ? VZ : 3) * g + (c - 3 * m), (ey & 1) * VP, VP - (ey & 1) * VP, VZ, m + 1);
            }
        }
        if (rxz & kAct) {
            const int lx = at(rxz);
            matrices();
            T v[P];
            Folded<P, T> f;
            auto put = [&](T *arr, int o, T lo, T hi) {
                arr[lx + o * SX] = lo;
                if (2 * o + 1 != Q) arr[lx + (Q - 1 - o) * SX] = hi;
            };
            line_read<P, SX>(A + lx, v);
            f.set(v);
            line_all<P, Q, -1>(Gf, f, [&](int o, T lo, T hi) { put(C, o, lo, hi); });
            if constexpr (!COLLOC) {
                line_all<P, Q, 1>(Bf, f, [&](int o, T lo, T hi) { put(A, o, lo, hi); });
                line_read<P, SX>(Bb + lx, v);
                f.set(v);
                line_all<P, Q, 1>(Bf, f, [&](int o, T lo, T hi) { put(Bb, o, lo, hi); });
            }
        }
        group_sync<NT>();
        // --- Z -----------------------------------------------------------------------------
        if (rxz >> 16 & kAct) {
            const int lz = at(rxz >> 16), az = rz & 15, bz = rz >> 4 & 15, gz = rz >> 8;
            matrices();
            T v[P];
            Folded<P, T> f;
            // [0]: the lane's points, o of u's lane and Q-1-o of r's; [1]: the other lane's
            T ur[2][NOH], us[2][NOH], ut[2][NOH];
            const T sg = vec ? T(-1) : T(1);
            auto split = [&](T (&u)[2][NOH], cptr<T> M, const T *arr, auto sym) {
                line_read<P, SZ>(arr + lz, v);
                f.set(v);
                line_halves<P, Q, decltype(sym)::value>(M, f, [&](int o, T E, T O, T) {
                    const T x = decltype(sym)::value > 0 ? E : O, y = decltype(sym)::value > 0 ? O : E;
                    u[0][o] = x + sg * y;
                    u[1][o] = x - sg * y;
                });
            };
            split(ut, Gf, A, std::integral_constant<int, -1>{});
            if constexpr (COLLOC) {
                const int l0 = vec ? lz + (Q - 1) * SZ : lz, l1 = vec ? lz : lz + (Q - 1) * SZ, st = vec ? -SZ : SZ;
#pragma unroll
                for (int o = 0; o < NOH; ++o) {
                    us[0][o] = Bb[l0 + o * st];
                    us[1][o] = Bb[l1 - o * st];
                    ur[0][o] = C[l0 + o * st];
                    ur[1][o] = C[l1 - o * st];
                }
            } else {
                split(us, Bf, Bb, std::integral_constant<int, 1>{});
                split(ur, Bf, C, std::integral_constant<int, 1>{});
            }
            ZLineGeom g;
            g.set(sC + gz * kTriCoef, sR[az], sR[bz]);
            const double wz = sR[Q + az] * sR[Q + bz];
            const int c0 = vec ? Q - 1 : 0, cs = vec ? -1 : 1;
            const int gx = STACK ? 0 : gz, gs = STACK ? gz : 0;
            gptr<T> out = (gptr<T>)a.g +
                          (pos.ex0 + gx + (int64_t)a.nex * (ey + (int64_t)a.ney * (pos.ez + gs))) * Q3 +
                          c0 * Q2 + bz * Q + az;
#pragma unroll
            for (int o = 0; o < NOH; ++o) {
                g.pin();
                double jr[3], js[3], r2[3], h[3], q[3];
                g.columns(sR[c0 + cs * o], jr, js);
                cross(jr, js, r2);
                const double f0 = wz * sR[Q + c0 + cs * o] * fast_rcp(dot3(g.jt, r2));
                double d = ur[0][o], e = us[0][o], t = ut[0][o];
#pragma unroll
                for (int k = 0; k < 3; ++k) h[k] = e * jr[k] - d * js[k];
                cross(g.jt, h, q);
#pragma unroll
                for (int k = 0; k < 3; ++k) q[k] += t * r2[k];
                d = lane_swap(ur[1][o]), e = lane_swap(us[1][o]), t = lane_swap(ut[1][o]);
#pragma unroll
                for (int k = 0; k < 3; ++k) h[k] = e * jr[k] - d * js[k];
                double q2[3];
                cross(g.jt, h, q2);
#pragma unroll
                for (int k = 0; k < 3; ++k) q2[k] += t * r2[k];
                double val = f0 * dot3(q, q2);
                asm volatile("" : "+v"(val));
                if (2 * o + 1 != Q || !vec) __builtin_nontemporal_store(val, out + cs * o * Q2);
            }
        }
        if (more) group_sync<NT>();
    }
}

}  // namespace mfhex
