// Tetrahedral P_p diffusion operator: the non-tensor basis path of Sec. 2.1 (libCEED) and
// Sec. 2.2 (its MAGMA / vendor-BLAS backend): the full basis-gradient matrix of one
// element is applied to all elements at once as a matrix product, here on
// the FP64 matrix cores.  Shared between the host set-up (tet.cpp) and the
// kernels (tet_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace mfhex {
namespace tet {

constexpr int kMaxP = 6;
constexpr int kComputeUnits = 256;
constexpr int n_basis(int p) { return (p + 1) * (p + 2) * (p + 3) / 6; }
constexpr int round_up(int n, int m) { return (n + m - 1) / m * m; }

// A set of three wavefronts takes the 48 tetrahedra of 8 hexahedra consecutive in x (three full
// 16-column tiles; pairs of hexahedra left a quarter of every tile empty).
constexpr int kCubes = 8;
constexpr int set_threads = 192;
constexpr int box_nodes(int p) { return (kCubes * p + 1) * (p + 1) * (p + 1); }

// Rows m of H (dim P_{p-1}) in tiles of four; the fragments of a tile: NS steps of the forward product,
// then 3 x NT of the transposed one, 64 doubles each.
constexpr int n_rows(int p) { return n_basis(p - 1); }
constexpr int tet_tiles(int p) { return (n_rows(p) + 3) / 4; }
constexpr int tet_tile_doubles(int p) { return (round_up(n_basis(p), 4) / 4 + 3 * (round_up(n_basis(p), 16) / 16)) * 64; }
constexpr int tet_frag_doubles(int p) { return tet_tiles(p) * tet_tile_doubles(p); }

// Fragments resident in LDS up to p = 4, streamed tile by tile above.  Sets per thread group share the
// fragments: two at p = 4 (three wavefronts per SIMD in two groups), four where they are streamed
// (twelve wavefronts, three on every SIMD).
constexpr bool tet_stream(int p) { return p >= 5; }
constexpr int tet_sets(int p) { return p <= 3 ? 1 : p == 4 ? 2 : 4; }
constexpr int tet_set_doubles(int p) { return (tet_stream(p) ? 1 : 2) * round_up(box_nodes(p), 2) + 48 * 6; }
constexpr size_t tet_lds(int p)
{
    return ((size_t)(tet_stream(p) ? 2 * tet_tile_doubles(p) : tet_frag_doubles(p)) +
            (size_t)tet_sets(p) * tet_set_doubles(p)) * 8;
}

// Sizes of one (p, q) instance: P basis functions, Q = q^3 points, padded to the matrix-core tile (points to 16,
// basis functions to 4 as a contraction extent and to 16 as an output extent).  They size the caller's workspace.
struct Dims {
    int p, q, P, Q, Qp, Pk, Pn;
};
constexpr Dims dims(int p, int q)
{
    return Dims{p, q, n_basis(p), q * q * q, round_up(q * q * q, 16), round_up(n_basis(p), 4), round_up(n_basis(p), 16)};
}

// Device tables:
//   frag [tile][NS + 3 NT][64]: lane l of forward step s holds H_d[4 tile + l%4][4 s + l/16], d = (l%16)/4 (0 for
//     d = 3); lane l of transposed step (d, t) holds H_d[4 tile + l/16][16 t + l%16] (0 outside the matrix)
//   fac [element][6]: |det J| J^-1 J^-T (xx, yy, zz, yz, xz, xy)
// Matrix-core operand layout of the 16x16x4 FP64 product D += A B (wave64): lane l supplies A[l%16][l/16] and
// B[l/16][l%16], and its result register r is D[4r + l/16][l%16] (checked on gfx950 with distinct entries).
struct TetLaunch {
    int p, nex, ney, nez, dirichlet;
    const int32_t *lattice;  // [P][4]: n1, n2, n3 of each basis function's node
    const double *frag, *fac;
    const double *x;
    double *y;
    hipStream_t stream;
};

struct TetSetupLaunch {
    int nex, ney;
    int64_t nelem;
    const double *vert;  // [(nex+1)(ney+1)(nez+1)][3]
    double *fac;
    int *bad;            // set to 1 when an element is degenerate
    hipStream_t stream;
};

hipError_t launch_tet_setup(const TetSetupLaunch &s);
hipError_t launch_tet_apply(const TetLaunch &a);

}  // namespace tet
}  // namespace mfhex
