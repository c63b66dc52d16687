// Tetrahedral P_p diffusion operator: set-up and fused apply kernels.
//
// Apply (Sec. 2.1 libCEED and Sec. 2.2 MAGMA: the non-tensor basis action as a matrix product over
// elements).  The elements are affine and the rule integrates the stiffness exactly, so the
// gradient of a P_p field, which lies in P_{p-1}, is taken in an orthonormal basis of P_{p-1}
// instead of at the q^3 points: with H_d[m][n] = int psi_m d phi_n / d xi_d the element stiffness is
//   K = sum_{ab} D_ab H_a^T H_b,   D = |det J| J^-1 J^-T (one symmetric 3x3 per element),
// M = p (p+1) (p+2) / 6 rows per direction in place of q^3 (10 of 27 at p = 3, 56 of 216 at p = 6),
// and six factors per element in place of six per point.
//
// A set of three wavefronts owns the 48 tetrahedra of 8 hexahedra consecutive in x, 16 columns each:
//   gather: the (8p+1)(p+1)^2 lattice nodes of the box once, coalesced, into LDS; each wavefront takes
//     its X (P x 16) from there as matrix-core B operands;
//   U = H X on the FP64 matrix cores, a tile = the three directions of four rows m: row 4 d + k of the
//     tile is H_d[4 t + k], so result register d of lane l holds d/dxi_d of row 4 t + l/16, element l%16,
//     and the 3x3 factor acts within a lane;
//   Y^T += V_d^T H_d: that register is the A operand of a 4-deep step over the same four rows, so the
//     products feed the transposed contraction with no data movement;
//   scatter: the element results are summed in LDS over the box, then one atomic per lattice node.
// The fragments of H (pre-swizzled, 64 consecutive doubles each) stay in LDS for the whole grid-stride
// run of a thread group at p <= 4 (46 KB at p = 4) and are streamed through two buffers, one tile ahead,
// shared by all its wavefronts, above (120 KB at p = 5, 273 KB at p = 6).
//
// Measured on MI355X, about 1e7 nodes, us an apply with its output fill, products at the q^3 points with
// per-point factors -> this form: p = 1..6 4626 -> 1908, 1221 -> 342, 1064 -> 285, 1019 -> 392,
// 1160 -> 446, 1579 -> 578.  The matrix cores alone need 72, 117, 138, 181, 249 us at p = 2..6; the
// rest is the scatter and the gather with their two barriers (p = 3), issue (VALU 21% busy) and, at
// p = 5, 6, three wavefronts a SIMD that wait for one another at every tile.
#include "mfhex_internal.h"
#include "tet.h"

namespace mfhex {
namespace tet {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ d4 mma(double a, double b, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Kuhn tetrahedron t: axis permutation; vertex k is the cube corner sum_{m<k} e_{pi[m]}.
__device__ __forceinline__ void kuhn_perm(int t, int &a0, int &a1, int &a2)
{
    const int perms[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
    a0 = perms[t][0];
    a1 = perms[t][1];
    a2 = perms[t][2];
}

// Blocks are dealt to the 8 XCDs round-robin; give each XCD a contiguous range of element groups.
__device__ __forceinline__ int64_t xcd_remap(int64_t bid, int64_t nb)
{
    const int64_t x = bid % kNumXcd, i = bid / kNumXcd;
    const int64_t q = nb / kNumXcd, r = nb % kNumXcd;
    return x * q + (x < r ? x : r) + i;
}

// fac[e][6] = |det J| J^-1 J^-T = adj(J) adj(J)^T / |det J| (xx, yy, zz, yz, xz, xy) of element e = 6 cube + t.
__global__ void k_tet_factors(int nex, int ney, int64_t nelem, const double *__restrict__ vert, double *__restrict__ fac,
                              int *__restrict__ bad)
{
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= nelem) return;
    double M[6];
    {
        const int64_t cube = e / 6;
        const int t = (int)(e % 6);
        const int ex = (int)(cube % nex), ey = (int)((cube / nex) % ney), ez = (int)(cube / ((int64_t)nex * ney));
        int a0, a1, a2;
        kuhn_perm(t, a0, a1, a2);
        int c[4][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {1, 1, 1}};
        c[1][a0] = 1;
        c[2][a0] = 1;
        c[2][a1] = 1;
        (void)a2;
        double X[4][3];
        for (int v = 0; v < 4; ++v) {
            const int64_t vid = (ex + c[v][0]) + (int64_t)(nex + 1) * ((ey + c[v][1]) + (int64_t)(ney + 1) * (ez + c[v][2]));
            for (int d = 0; d < 3; ++d) X[v][d] = vert[3 * vid + d];
        }
        double Jm[3][3];  // J[row = physical dir][col = reference dir]
        for (int r = 0; r < 3; ++r)
            for (int cc = 0; cc < 3; ++cc) Jm[r][cc] = X[cc + 1][r] - X[0][r];
        // adjugate: adj(J)[i][k] = cofactor(J)[k][i]
        double A[3][3];
        for (int i = 0; i < 3; ++i)
            for (int k = 0; k < 3; ++k) {
                const int r0 = (k + 1) % 3, r1 = (k + 2) % 3, c0 = (i + 1) % 3, c1 = (i + 2) % 3;
                A[i][k] = Jm[r0][c0] * Jm[r1][c1] - Jm[r0][c1] * Jm[r1][c0];
            }
        const double det = Jm[0][0] * A[0][0] + Jm[0][1] * A[1][0] + Jm[0][2] * A[2][0];
        if (!(det != 0.0) || !isfinite(det)) bad[0] = 1;
        const double s = 1.0 / fabs(det);
        // (adj adj^T)[a][b] = sum_i adj[a][i] adj[b][i]
        auto aa = [&](int x, int y) { return (A[x][0] * A[y][0] + A[x][1] * A[y][1] + A[x][2] * A[y][2]) * s; };
        M[0] = aa(0, 0);
        M[1] = aa(1, 1);
        M[2] = aa(2, 2);
        M[3] = aa(1, 2);
        M[4] = aa(0, 2);
        M[5] = aa(0, 1);
    }
    for (int f = 0; f < 6; ++f) fac[6 * e + f] = M[f];
}

// Node slot i of the box: coordinates (bx, by, bz) in [0, 8p] x [0, p] x [0, p], or (ALONG_Y: its hexahedra consecutive in
// y, for rows that would fill a quarter of it at most) [0, p] x [0, 8p] x [0, p].
template <int p, bool ALONG_Y>
struct Box {
    static constexpr int L = kCubes * p + 1, BX = ALONG_Y ? p + 1 : L, BY = ALONG_Y ? L : p + 1, NB = BX * BY * (p + 1);
    __device__ static __forceinline__ void coords(int i, int &bx, int &by, int &bz)
    {
        bx = i % BX;
        by = (i / BX) % BY;
        bz = i / (BX * BY);
    }
};

// Box position of basis function n of column j (tetrahedron j % 6 of hexahedron j / 6).
template <int p, bool ALONG_Y>
__device__ __forceinline__ int box_node(int j, const int32_t *__restrict__ lattice, int n)
{
    int a0, a1, a2;
    kuhn_perm(j % 6, a0, a1, a2);
    (void)a2;
    const int n1 = lattice[4 * n], n2 = lattice[4 * n + 1], n3 = lattice[4 * n + 2];
    // lattice offset n1 v1 + n2 v2 + n3 v3 with v1 = e_a0, v2 = e_a0 + e_a1, v3 = (1,1,1)
    int a[3] = {n3, n3, n3};
    a[a0] += n1 + n2;
    a[a1] += n2;
    a[ALONG_Y ? 1 : 0] += (j / 6) * p;
    using B = Box<p, ALONG_Y>;
    return a[0] + B::BX * (a[1] + B::BY * a[2]);
}

template <int p, bool ALONG_Y>
__global__ void __launch_bounds__(set_threads * tet_sets(p))
k_tet_apply(const int ngx, const int nex, const int ney, const int nez, const int dirichlet, const int per,
            const int32_t *__restrict__ lattice, const double *__restrict__ frag, const double *__restrict__ fac,
            const double *__restrict__ x, double *__restrict__ y)
{
    using B = Box<p, ALONG_Y>;
    constexpr int P = n_basis(p), T = tet_tiles(p), NS = round_up(P, 4) / 4, NT = round_up(P, 16) / 16;
    constexpr int FT = tet_tile_doubles(p), SETS = tet_sets(p), NTH = set_threads * SETS;
    constexpr bool STREAM = tet_stream(p);
    constexpr int NB = B::NB, R = (NB + set_threads - 1) / set_threads;
    extern __shared__ __align__(16) double smem[];
    const int tid = threadIdx.x, set = tid / set_threads, t3 = tid - set * set_threads;
    const int lane = t3 & 63, wave = t3 >> 6, el = lane & 15, kq = lane >> 4;
    double *const sF = smem;
    // per set: input and output boxes (one and the same where the fragments are streamed: there LDS is short, and
    // the products are long enough to hide two more barriers), then the factors of its 48 columns
    double *const xb = sF + (STREAM ? 2 : T) * FT + set * tet_set_doubles(p);
    double *const yb = STREAM ? xb : xb + round_up(NB, 2), *const sD = yb + round_up(NB, 2);

    // LDS positions of this lane's operands: X[4 s + kq][column 16 wave + el], and result register r of output
    // tile t: element 4 r + kq, basis function 16 t + el (65535: no basis function)
    uint32_t xa[(NS + 1) / 2], ya[NT * 2];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int n = 4 * s + kq;
        const uint32_t v = n < P ? (uint32_t)box_node<p, ALONG_Y>(16 * wave + el, lattice, n) : 65535u;
        if (s & 1) xa[s / 2] |= v << 16;
        else xa[s / 2] = v;
    }
#pragma unroll
    for (int i = 0; i < NT * 4; ++i) {
        const int n = 16 * (i / 4) + el, j = 16 * wave + 4 * (i % 4) + kq;
        const uint32_t v = n < P ? (uint32_t)box_node<p, ALONG_Y>(j, lattice, n) : 65535u;
        if (i & 1) ya[i / 2] |= v << 16;
        else ya[i / 2] = v;
    }
    auto half = [](uint32_t v, int i) {
        asm volatile("" : "+v"(v));  // unpacked at each use, not held unpacked
        return i & 1 ? v >> 16 : v & 65535u;
    };

    const int nx = p * nex + 1, ny = p * ney + 1, nz = p * nez + 1;
    const int ngy = ALONG_Y ? (ney + kCubes - 1) / kCubes : ney;
    const int64_t nsteps = (int64_t)ngx * ngy * nez;
    // contiguous runs of steps, y fastest (neighbours in y share the largest faces)
    const int64_t first = (xcd_remap(blockIdx.x, gridDim.x) * SETS + set) * per;
    struct Step {
        int64_t node, elem;  // first lattice node, first element
        int ncols, cx, ey, ez;
        bool on, edge;       // edge: some node may be masked or outside the mesh
    };
    auto step_at = [&](int i) {
        Step q;
        const int64_t s = first + i;
        q.on = i < per && s < nsteps;
        const unsigned u = (unsigned)(q.on ? s : 0);
        const int gy = (int)(u % (unsigned)ngy);
        const unsigned v = u / (unsigned)ngy;
        const int gx = (int)(v % (unsigned)ngx);
        q.ez = (int)(v / (unsigned)ngx);
        q.cx = ALONG_Y ? gx : gx * kCubes;
        q.ey = ALONG_Y ? gy * kCubes : gy;
        const int left = ALONG_Y ? ney - q.ey : nex - q.cx, nc = left < kCubes ? left : kCubes;
        q.ncols = 6 * nc;
        q.node = (int64_t)p * (q.cx + (int64_t)nx * (q.ey + (int64_t)ny * q.ez));
        q.elem = 6 * (q.cx + (int64_t)nex * (q.ey + (int64_t)ney * q.ez));
        q.edge = nc < kCubes || (dirichlet && (gx == 0 || gx == ngx - 1 || gy == 0 || gy == ngy - 1 || q.ez == 0 ||
                                               q.ez == nez - 1));
        return q;
    };
    // Node slots of this lane: their offsets from a step's first node are the same in every step (32 bits: N < 2^31),
    // kept in registers where there are few of them.
    constexpr int RK = STREAM ? 1 : R;
    uint32_t offs[RK];
    auto offset_of = [&](int r) {
        int bx, by, bz, i = t3 + r * set_threads;
        asm volatile("" : "+v"(i));  // recomputed at each use: kept, they would spill
        B::coords(i, bx, by, bz);
        return (uint32_t)bx + (uint32_t)nx * ((uint32_t)by + (uint32_t)ny * (uint32_t)bz);
    };
#pragma unroll
    for (int r = 0; r < RK; ++r) offs[r] = offset_of(r);
    auto slot = [&](const Step &q, int r, uint32_t &off) {  // false where masked or outside the mesh
        off = STREAM ? offset_of(r) : offs[STREAM ? 0 : r];
        bool ok = q.on && t3 + r * set_threads < NB;
        if (q.edge) {
            int bx, by, bz, i = t3 + r * set_threads;
            asm volatile("" : "+v"(i));
            B::coords(i, bx, by, bz);
            const int I = p * q.cx + bx, J = p * q.ey + by, K = p * q.ez + bz;
            ok = ok && (ALONG_Y ? J < ny : I < nx) && !(dirichlet && (I == 0 || I == nx - 1 || J == 0 || J == ny - 1 || K == 0 || K == nz - 1));
        }
        return ok;
    };
    double xs[R];
    d2 fd = {0.0, 0.0};
    auto load = [&](const Step &q) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t off;
            xs[r] = slot(q, r, off) ? (x + q.node)[off] : 0.0;
        }
        // factors of the set's columns (none past the row's end: those columns' results are dropped)
        if (q.on && t3 < 3 * q.ncols) fd = reinterpret_cast<const d2 *>(fac + 6 * q.elem)[ALONG_Y ? t3 / 18 * (int64_t)(18 * nex) + t3 % 18 : t3];
    };

    constexpr int RF = (FT + NTH - 1) / NTH;  // streamed fragments: a tile's share of one lane
    double stage[STREAM ? RF : 1];
    auto stage_load = [&](int tile) {
#pragma unroll
        for (int k = 0; k < RF; ++k)
            if (tid + k * NTH < FT) stage[k] = frag[(size_t)tile * FT + tid + k * NTH];
    };
    auto stage_store = [&](int buf) {
#pragma unroll
        for (int k = 0; k < RF; ++k)
            if (tid + k * NTH < FT) sF[buf * FT + tid + k * NTH] = stage[k];
    };
    int buf = 0;
    if constexpr (STREAM) {
        stage_load(0);
        stage_store(0);
    } else {
        for (int i = tid; i < T * FT; i += NTH) sF[i] = frag[i];
    }

    Step q = step_at(0);
    load(q);
    for (int it = 0; it < per; ++it) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (t3 + r * set_threads < NB) {
                xb[t3 + r * set_threads] = xs[r];
                if (!STREAM) yb[t3 + r * set_threads] = 0.0;
            }
        if (t3 < 3 * 48) reinterpret_cast<d2 *>(sD)[t3] = fd;
        __syncthreads();
        double xf[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint32_t v = half(xa[s / 2], s);
            xf[s] = v != 65535u ? xb[v != 65535u ? v : 0] : 0.0;
        }
        if constexpr (STREAM) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (t3 + r * set_threads < NB) yb[t3 + r * set_threads] = 0.0;
        }
        const d2 *const dcol = reinterpret_cast<const d2 *>(sD) + 3 * (16 * wave + el);
        d2 f0, f1, f2;
        if constexpr (!STREAM) f0 = dcol[0], f1 = dcol[1], f2 = dcol[2];
        const Step cur = q;
        q = step_at(it + 1);
        if (!STREAM && it + 1 < per) load(q);  // travels behind the products
        d4 yacc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) yacc[t] = d4{0.0, 0.0, 0.0, 0.0};
        // one tile: fragments U at a time, the next U in flight (all at once would not fit the registers)
        auto tile = [&](const double *F) {
            constexpr int S = NS + 3 * NT, U = STREAM ? 2 : 4, NG = (S + U - 1) / U;
            double fr[2][U], v[3];
            d4 u = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < U; ++k) fr[0][k] = k < S ? F[k * 64 + lane] : 0.0;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if ((g + 1) * U + k < S) fr[(g + 1) & 1][k] = F[((g + 1) * U + k) * 64 + lane];
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const int i = g * U + k;
                    if (i < NS) u = mma(fr[g & 1][k], xf[i < NS ? i : 0], u);
                    if (i == NS) {
                        if constexpr (STREAM) f0 = dcol[0], f1 = dcol[1], f2 = dcol[2];
                        const double xx = f0[0], yy = f0[1], zz = f1[0], yz = f1[1], xz = f2[0], xy = f2[1];
                        v[0] = xx * u[0] + xy * u[1] + xz * u[2];
                        v[1] = xy * u[0] + yy * u[1] + yz * u[2];
                        v[2] = xz * u[0] + yz * u[1] + zz * u[2];
                    }
                    if (i >= NS && i < S) yacc[(i - NS) % NT] = mma(v[(i - NS) / NT], fr[g & 1][k], yacc[(i - NS) % NT]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if constexpr (STREAM) {
            // (the barrier after the first tile also separates clearing the box from adding to it)
            static_assert(T > 1, "a barrier before the box is added to");
            for (int t = 0; t < T; ++t) {
                stage_load(t + 1 < T ? t + 1 : 0);
                tile(sF + buf * FT);
                buf ^= 1;
                stage_store(buf);
                __syncthreads();  // the next tile's fragments are in; this tile's may be overwritten
            }
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t) tile(sF + t * FT);
        }
        if (cur.on) {
#pragma unroll
            for (int i = 0; i < NT * 4; ++i) {
                const uint32_t v = half(ya[i / 2], i);
                if (v != 65535u && 16 * wave + 4 * (i % 4) + kq < cur.ncols) atomicAdd(&yb[v], yacc[i / 4][i % 4]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t off;
            if (slot(cur, r, off)) unsafeAtomicAdd(y + cur.node + off, yb[t3 + r * set_threads]);
        }
        if (STREAM && it + 1 < per) load(q);
    }
}

template <int p, bool ALONG_Y>
hipError_t apply_box(const TetLaunch &a)
{
    constexpr size_t lds = tet_lds(p);
    static_assert(lds <= 163840, "LDS of a thread group");
    auto kern = k_tet_apply<p, ALONG_Y>;
    if (lds > 65536) {
        const hipError_t e =
            hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    // one resident round of thread groups, each with a contiguous share of the steps
    const int ngx = ALONG_Y ? a.nex : (a.nex + kCubes - 1) / kCubes, ngy = ALONG_Y ? (a.ney + kCubes - 1) / kCubes : a.ney;
    const int64_t nsteps = (int64_t)ngx * ngy * a.nez;
    static const int resident = [&] {
        int n = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, set_threads * tet_sets(p), lds) == hipSuccess && n > 0
                   ? n
                   : 1;
    }();
    const int64_t sets = (int64_t)kComputeUnits * resident * tet_sets(p);
    const int64_t per = (nsteps + sets - 1) / sets;
    const int64_t nset = (nsteps + per - 1) / per, nblk = (nset + tet_sets(p) - 1) / tet_sets(p);
    hipLaunchKernelGGL(kern, dim3((unsigned)nblk), dim3(set_threads * tet_sets(p)), lds, a.stream, ngx, a.nex, a.ney,
                       a.nez, a.dirichlet, (int)per, a.lattice, a.frag, a.fac, a.x, a.y);
    return hipGetLastError();
}

// Boxes along x, whose rows of nodes are long, unless the row fills a quarter of one at most and a column of elements
// fills more: 2e6 nodes, p = 1, 4, 5, 6, rows of one 1346, 459, 491, 628 us along x, of two 1029, 263, 306, 398.
template <int p>
hipError_t apply_p(const TetLaunch &a)
{
    const int64_t pad = (a.ney + kCubes - 1) / kCubes * kCubes;
    return 4 * a.nex <= kCubes && pad * a.nex < (int64_t)kCubes * a.ney ? apply_box<p, true>(a) : apply_box<p, false>(a);
}

}  // namespace

hipError_t launch_tet_setup(const TetSetupLaunch &s)
{
    hipLaunchKernelGGL(k_tet_factors, dim3((unsigned)((s.nelem + 127) / 128)), dim3(128), 0, s.stream, s.nex, s.ney,
                       s.nelem, s.vert, s.fac, s.bad);
    return hipGetLastError();
}

hipError_t launch_tet_apply(const TetLaunch &a)
{
    switch (a.p) {
    case 1: return apply_p<1>(a);
    case 2: return apply_p<2>(a);
    case 3: return apply_p<3>(a);
    case 4: return apply_p<4>(a);
    case 5: return apply_p<5>(a);
    case 6: return apply_p<6>(a);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace tet
}  // namespace mfhex
