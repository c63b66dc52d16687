// Internal declarations shared by the host runtime (*.cpp) and the kernels (*.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <string>

#include "../../include/mfhex.h"

namespace mfhex {

constexpr int kMaxP = 9;   // nodes per direction (p = 8)
constexpr int kMaxQ = 10;  // quadrature points per direction (q = p + 2)
constexpr int kQdDiff = 6; // symmetric geometric factors per point (Voigt rr, ss, tt, st, rt, rs)
constexpr int kNumXcd = 8; // MI355X: 8 accelerator complex dies, blocks dealt round-robin

// 1D data of one operator, FP64 (host master copy) and FP32.
struct Basis1D {
    int P = 0, Q = 0;
    bool colloc = false;             // Q == P and points == nodes (B = I)
    double nodes[kMaxP];             // Gauss-Lobatto nodes
    double xq[kMaxQ], wq[kMaxQ];     // quadrature points / weights
    double B[kMaxQ * kMaxP];         // B[a*P + i] = l_i(xq_a)
    double D[kMaxQ * kMaxQ];         // D[a*Q + b] = derivative at point a of the Lagrange
                                     // polynomial through the points that is 1 at point b
    double Gn[kMaxQ * kMaxP];        // Gn[a*P + i] = l_i'(xq_a)   (direct, for checks)
};

// Host side of the basis construction (basis.cpp).
int build_basis(int p, int q, int quad, Basis1D *out, std::string *err);
int gauss_rule(int n, double *x, double *w);
int lobatto_rule(int n, double *x, double *w);

// Kernel arguments common to the operator kernels.
struct OpView {
    int64_t nelem;
    int32_t nex, ney, nez, p, q;
    int64_t nnodes;
    const int32_t *offsets;  // [E][P^3], -1 = masked node
    const void *qdata;       // [E][g][Q^3] in the apply precision
    const double *kappa;     // [E][Q^3] or null
};

enum Mode : int { kMass = 0, kDiff = 1, kRhs = 2 };

// Launch configuration of the apply: the variant (elements and threads per
// thread group, vectors per chunk) and, for the mass operator, the number of
// consecutive element groups one thread group pipelines through.
constexpr int kMaxChain = 64;
struct LaunchCfg {
    int variant = 0;
    int chain = 0;  // pipeline depth; 0: automatic (pipeline_depth)
};

struct ApplyLaunch {
    OpView v;
    int P, colloc;
    const void *basis_dev; // device basis block (B, B^T, D, D^T) in the apply precision
    const double *basis64; // the same block in FP64
    int dirichlet;
    int prec;             // MFHEX_F64 / MFHEX_F32
    int mode;             // kMass / kDiff / kRhs
    int vark;             // multiply the factors by kappa
    int nvec;
    int variant;          // launch variant (elements and threads per group)
    int chain;            // mass: element groups per thread group (software pipeline depth), >= 1
    int otf;              // diffusion FP64: geometric factors evaluated in the kernel from the vertices
    const double *vert;   // device vertex coordinates [(nex+1)(ney+1)(nez+1)][3] (line-fused kernels)
    const void *x;        // input (for kRhs: the per-point f, FP64)
    void *y;              // output (accumulated)
    const double *wdet;   // kRhs: w*detJ per point
    void *ebuf;           // deterministic scatter: element values [E][P^3][nvec] (null: atomics into y)
    hipStream_t stream;
};

// Diagonal of the assembled operator (FP64), accumulated into d.
struct DiagLaunch {
    OpView v;  // FP64 factors
    int P, colloc, mode, vark;
    const double *basis_dev;
    double *d;
    hipStream_t stream;
};

struct KgradLaunch {
    OpView v;
    int P, colloc;
    const double *basis_dev, *vert;
    const double *u, *r;
    double *g;
    int dirichlet;
    hipStream_t stream;
};

// LDS layout of one element's working array: [c][b][a] with an odd row pitch so
// that pencils along any axis hit distinct banks; q = 10 keeps the pitch of 10,
// which fits a split group's four arrays in 32 KB, five groups per CU (4% faster
// than pitch 11 for the prefetching split group in same-box A/B, where the
// padding left room for four).
constexpr int lds_pitch(int Q) { return (Q % 2 == 0 && Q != 10) ? Q + 1 : Q; }
constexpr int lds_buf(int Q) { return lds_pitch(Q) * Q * Q; }
constexpr int apply_nbuf(int mode, bool split = false) { return mode == 1 ? (split ? 4 : 3) : 1; }
// Split stages of the diffusion kernel: with G elements and one vector per
// group of NT >= 256 threads whose widest contraction (G Q^2 lines) fits in
// half the group, the two halves (two wavefronts each) share every contraction:
// each takes half of the output rows, and independent contractions run side
// by side, so no wavefront of the group sits out a contraction stage.  A
// fourth LDS array lets every such stage write a different array than it
// reads.  (Measured on MI355X: 2% faster at q = 10 with 256 threads; with 128
// threads the extra registers cost one wave per SIMD and 6% at q = 8.)
constexpr bool split_stages(int Q, int mode, int G, int NT, int VC)
{
    return mode == 1 && VC == 1 && NT >= 256 && 2 * G * Q * Q <= NT;
}

// Launch variants of the fused kernels for q points per direction: G elements per thread group of NT
// threads.  Which kernel a number stands for depends on the operator (line_variant below): the line-fused
// kernel takes 9 .. 14 of diffusion with Gauss points, and 0 .. 4 of collocated (but elem_slot) or in-kernel-factor
// diffusion and of mass with Gauss points.  Variants 0 .. 4 of the other operators carry one vector at a
// time through the element with stored factors (rows: Q = 2 .. 10); 5 .. 8 carry a chunk of VC = 2, 4, 8,
// 16 vectors of a multi-vector together (one element per group; 6 and 7 of collocated diffusion in k_mline where
// mline_serves says so), sharing the geometric factors and reading
// / writing each node's chunk as one contiguous run; 15 and 16 are chunks of 4 and 8 vectors whose
// collocated gradient contractions run on the FP64 matrix cores.
constexpr int kNumVariants = 17;
// At q = 6 and 7 variant 4 fills the lanes: every contraction of the diffusion
// kernel runs over G q^2 lines (q^2 = 36, 49), so 7 and 5 elements per
// 256-thread group give 252 and 245 lines, where groups of 1 or 2 elements
// leave 44-62% of the lanes idle.
// Late factor loads: at q = 7 and 9 variant 2 and at q = 8 and 10 variants 4 and 2 load each
// point's geometric factors in the pointwise stage (the listed number of points at a time)
// instead of at the start of the element group.  The prefetched factors of a lane's points hold
// 6 x 2 registers per point (8 points per lane at q = 10 with 128 threads: 96 registers) through
// every forward contraction; loaded late they are live in the pointwise stage only, so more
// wavefronts fit on a SIMD (q = 7..9, two points at a time: 64-72 registers instead of 120-142)
// while the loads' latency is no longer hidden by the contractions.  At q = 10 this was 6% faster
// on one box and 5% slower on another against variant 0 with 128 threads.  With 256 threads
// (split stages) the late loads are the fastest stored-factor launches at q = 9 and 10: 68 and 81 registers instead of 101
// and 126, so that five to six groups fit per CU (at q = 10 with the unpadded row pitch, which
// puts the four arrays of a group in 32 KB); same-box A/B, one element per group: q = 9 6%
// faster than the best prefetching variant, q = 10 11%.
constexpr int kVarG[9][5] = {
    {16, 8, 32, 16, 32}, {8, 4, 16, 8, 16}, {4, 2, 8, 4, 8}, {4, 2, 5, 2, 8}, {1, 3, 1, 2, 7},
    {1, 2, 1, 4, 5},     {1, 2, 1, 2, 1},   {2, 1, 1, 1, 1}, {1, 1, 1, 1, 2}};
constexpr int kVarNT[9][5] = {
    {64, 64, 64, 128, 128},  {64, 64, 64, 128, 128},  {64, 64, 64, 128, 128},
    {128, 64, 256, 128, 256}, {64, 256, 128, 128, 256}, {64, 128, 64, 256, 256},
    {128, 256, 64, 128, 128}, {256, 128, 128, 256, 256}, {256, 128, 128, 256, 256}};
// points per factor-load batch in the pointwise stage (0: factors prefetched at the group start)
constexpr int kVarLate[9][5] = {{0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}, {0, 0, 2, 0, 0}, {0, 2, 0, 0, 0},
                                {0, 0, 3, 3, 0}, {0, 2, 0, 0, 2}, {0, 0, 2, 0, 2}, {0, 0, 4, 2, 0}};
constexpr int variant_late(int Q, int v) { return v < 5 ? kVarLate[Q - 2][v] : 0; }
// of those, points per lane whose factors are still prefetched at the group start (the rest load late)
constexpr int kVarPre[9][5] = {{0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}, {0, 0, 0, 0, 0},
                               {0, 0, 3, 3, 0}, {0, 0, 0, 0, 2}, {0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}};
constexpr int variant_pre(int Q, int v) { return v < 5 ? kVarPre[Q - 2][v] : 0; }
constexpr bool variant_mx(int v) { return v >= 15; }
constexpr int variant_vc(int v)
{
    return v == 15 ? 4 : v == 16 ? 8 : v < 5 || v >= 9 ? 1 : v == 5 ? 2 : v == 6 ? 4 : v == 7 ? 8 : 16;
}
// The line-fused kernel (k_line, line_kernels.hpp): variants 9 .. 14 of the diffusion operator with
// Gauss points, and variants 0 .. 4 of the collocated diffusion, the in-kernel-factor (OTF) and the
// mass operator with Gauss points.  G q^2 lines in the widest stage, one per lane, so the slots take
// the (elements, threads) pairs that leave few lanes idle.
constexpr int kLineG[9][5] = {{16, 32, 8, 64, 4}, {7, 14, 28, 4, 2}, {4, 8, 16, 2, 1}, {5, 10, 2, 4, 1}, {7, 3, 5, 1, 2},
                              {5, 1, 2, 4, 3},    {2, 1, 4, 3, 1},   {3, 1, 2, 1, 3},  {1, 3, 2, 1, 2}};
constexpr int line_nt(int Q, int G) { return (G * Q * Q + 63) / 64 * 64; }
// Elements a line-fused group marches through where no depth was asked for: at most `most`, and no more than leave
// four rounds of resident groups on the chip (16384 wavefronts), since a march trades parallelism for carried faces.
// (Diffusion, p = 3, 5, 7 at 1e7 nodes: 2, 4 and 8 within 3%, 16 up to 10% slower.)
constexpr int kMarchDiff = 8;
constexpr int line_march(int most, int ney, int64_t columns, int nt)
{
    const int64_t m = columns * ney * (nt / 64) / 16384, cap = most < ney ? most : ney;
    return (int)(m < 1 ? 1 : m < cap ? m : cap);
}
constexpr int line_slot(int v) { return v < 5 ? v : v == 14 ? 0 : v - 9; }
// Collocated diffusion in FP64, of the numbers 0 .. 4 the one that is the element-at-a-time kernel with stored factors instead
// (k_apply, in the shape of kElemShape; elem_slot, -1: none), at the q where it is the faster one somewhere (kElemColl).
constexpr int kElemSlotColl[9] = {3, -1, -1, -1, -1, -1, -1, 4, -1};
constexpr int kElemShape[9] = {0, 0, 0, 4, 4, 4, 0, 4, 3};
constexpr int elem_slot(int Q, int mode, bool colloc, bool otf, bool f32)
{
    return mode == 1 && colloc && !otf && !f32 ? kElemSlotColl[Q - 2] : -1;
}
// The variant whose group shape (variant_g, variant_nt below) an element-at-a-time launch takes.
constexpr int elem_shape(int Q, int mode, bool colloc, bool otf, bool f32, int v)
{
    return v == elem_slot(Q, mode, colloc, otf, f32) ? kElemShape[Q - 2] : v;
}
constexpr bool line_variant(int Q, int mode, bool colloc, bool otf, bool f32, int v)
{
    if (mode == 0) return v < 5 && !colloc;
    return mode == 1 && v != elem_slot(Q, mode, colloc, otf, f32) && (colloc || otf ? v < 5 : v >= 9 && v <= 14);
}
// Collocated diffusion, several vectors: variants 6 and 7 are the line-fused multi-vector kernel (k_mline) with chunks
// of 4 and 8 vectors; G q^2 VC lanes.  G fills the last wavefront (q <= 5) while two groups fit a CU's LDS.
constexpr bool mline_variant(int mode, bool colloc, int v) { return mode == 1 && colloc && (v == 6 || v == 7); }
constexpr int mline_g(int Q, int v)
{
    return v == 7 ? (Q == 2 ? 8 : Q == 3 ? 3 : Q == 4 ? 2 : Q == 5 ? 2 : 1) : (Q == 2 ? 16 : Q == 3 ? 7 : Q == 4 ? 4 : Q == 5 ? 2 : 1);
}
constexpr int mline_nt(int Q, int v) { return (mline_g(Q, v) * Q * Q * (v == 7 ? 8 : 4) + 63) / 64 * 64; }
// Elements of a coefficient gradient group (q = 2 .. 10), two lanes per z-line: the lanes of a wavefront filled at low q
// (q = 5, 6 Gauss, G = 5, 3 against 2, 1: 129, 327 against 155, 395 us at 3e6 and 1e7 nodes); from q = 7 one element,
// whose two or three wavefronts hide more than a larger group's fuller ones (q = 7: 109 us, 163 with G = 3; q = 9: 70,
// 103 with G = 2).
constexpr int kKgradG[9] = {8, 7, 4, 5, 3, 1, 1, 1, 1};
constexpr int kgrad_g(int Q) { return kKgradG[Q - 2]; }
constexpr bool variant_gf(int v) { return v >= 9 && v <= 14; }
// The mass operator keeps one LDS array per element instead of three and has
// far less work per element, so at low order its single-vector variants
// carry more elements per group.
constexpr int mass_group_scale(int Q) { return Q <= 4 ? 4 : Q <= 6 ? 2 : 1; }
constexpr int variant_g(int Q, int v, int mode = 1)
{
    return v < 5 ? kVarG[Q - 2][v] * (mode == 1 ? 1 : mass_group_scale(Q)) : 1;
}
constexpr int variant_nt(int Q, int v)
{
    return v < 5 ? kVarNT[Q - 2][v]
                 : (Q * Q * variant_vc(v) <= 64 ? 64 : Q * Q * variant_vc(v) <= 128 ? 128 : 256);
}
// Dynamic LDS bytes of one group of the fused apply.
constexpr bool variant_split(int Q, int v, int mode)
{
    return split_stages(Q, mode, variant_g(Q, v, mode), variant_nt(Q, v), variant_vc(v));
}
// Multi-vector chunks of the diffusion kernel add their results to y in runs of at least 64 bytes
// per node (8 FP64 or 16 FP32 vectors) when a launch has more vectors than one chunk: y is
// node-major, and a chunk of fewer vectors would leave partly written lines in the L2 between
// chunks, which go back to HBM as 32-byte partial writes.  The element values of all but the last
// chunk of a run wait in LDS ([P^3][run - VC]), next to the element's restriction offsets ([P^3]
// int32).  A launch whose vectors fit one chunk adds them directly.
constexpr int scatter_run(int vc, int elem_bytes) { return vc * elem_bytes >= 64 ? vc : 64 / elem_bytes; }
constexpr bool staged_scatter(int mode, int vc, int elem_bytes)
{
    return mode == 1 && vc > 1 && scatter_run(vc, elem_bytes) > vc;
}
constexpr size_t apply_lds(int P, int Q, int mode, int elem_bytes, int v, bool stage = false)
{
    const int vc = variant_vc(v);
    const size_t p3 = (size_t)P * P * P;
    return (size_t)variant_g(Q, v, mode) * vc * apply_nbuf(mode, variant_split(Q, v, mode)) * lds_buf(Q) * elem_bytes +
           (stage && staged_scatter(mode, vc, elem_bytes) ? p3 * (scatter_run(vc, elem_bytes) - vc) * elem_bytes + p3 * 4
                                                          : 0);
}
// Largest dynamic LDS of one thread group (gfx950 has 160 KB per CU; above 64 KB the kernel is
// launched with a raised limit).  96 KB admits 8-vector chunks at q = 7, 4-vector chunks at q = 9
// and 16-vector chunks at q = 6 while still leaving room for a second group on the CU.
constexpr size_t kMaxLds = 98304;
constexpr size_t kLdsTwoGroups = 81920;  // at most this much LDS leaves room for two thread groups per CU
// Rows (index q - 2) from which k_mline's groups are faster than k_apply's single elements, in chunks of 4 with 2 or 4
// vectors and with 3 (k_apply has no chunk of three), and in chunks of 8; us of 3e5 nodes, k_apply and k_mline:
//   FP64, chunks of 4, 2 vectors: p = 1 rows of 1, 2, 3 52 95, 75 97, 0.91; p = 2 rows of 1, 2, 3, 4 18 39, 20 32, 22 25,
//     0.99; p = 3 rows of 1, 2, 3 12 25, 16 20, 0.99; 4 vectors: p = 4 rows of 1, 2 17 19, 0.89; 3 vectors: p = 2, 3 rows of
//     one 30 40, 20 26
//   FP64, chunks of 8, 8 vectors: p = 2 rows of 1, 2 41 48, 0.85; p = 3 29 32, 0.83; p = 4 rows of 1, 2, 3, 4 26 38, 31 34,
//     35 42, 35 39 (5 vectors 1.21, 0.90, 1.10, 0.94)
//   FP32, chunks of 8, 8 vectors: p = 1 rows of 1, 2, 3 52 76, 71 83, 0.88; p = 4 rows of 1, 2 17 22, 0.95
constexpr int kMlineRows4[9] = {3, 4, 3, 2, 1, 1, 1, 1, 1};
constexpr int kMlineRows3[9] = {2, 2, 2, 1, 1, 1, 1, 1, 1};
constexpr int kMlineRows8[9] = {2, 2, 2, 4, 1, 1, 1, 1, 1};
constexpr int kMlineRows8f32[9] = {3, 2, 1, 2, 1, 1, 1, 1, 1};
// Sizes whose stored factors come from the Infinity Cache, where k_apply's single elements are ahead of k_mline's groups
// (MB): p = 4, 8 .. 12 FP64 vectors, 16^3 elements (25 MB) 34 and 68 us against 36 and 74, 21^3 (56 MB), 12 vectors 0.82;
// p = 5, 2 FP32 vectors, 17^3 and 21^3 (48 MB) 23 and 39 against 26 and 43, 29^3 (126 MB) 0.95; p = 6, 2 and 4, 11^3 (11 MB)
// 14 and 17 against 15 and 18, 14^3 (23 MB) 25 against 22.
constexpr int cached_factors_mb(int Q, int elem_bytes) { return elem_bytes == 8 ? (Q == 5 ? 32 : 0) : Q == 6 ? 64 : Q == 7 ? 16 : 0; }
constexpr bool cached_factors(int Q, int elem_bytes, int64_t nelem)
{
    return nelem * (Q * Q * Q * kQdDiff * elem_bytes) <= (int64_t)cached_factors_mb(Q, elem_bytes) << 20;
}
constexpr int64_t kFewElements = 256;  // at most an element a compute unit
// Whether k_mline takes a launch of nvec vectors in chunks of variant v (else k_apply), by the row length, the size of the
// stored factors and the chunks:
// - rows as above (with more than 14 vectors in 8s from rows of one on, at p = 4 of two), and sizes;
// - k_apply works through the chunks of an element in turn, k_mline's are groups of their own: with few elements they fill
//   the chip (p = 7, 64 elements, 12 vectors 22 us, 12);
// - chunks of less than 64 bytes a node update half a line at a time, which k_apply avoids by staging two chunks where two
//   of its groups fit a CU.  Several such chunks stay with k_mline in FP32 where its stages are that much shorter (p = 1
//   and p >= 6, 9 to 48 vectors: 0.35 to 1.0 of k_apply's time; p = 2: 0.6 to 0.98, but 16, 32, 48 up to 1.17 at 3e4 nodes),
//   and at p = 3 .. 5 where their number is odd, so that k_apply's last run is half empty, and the last is full (24 and 40
//   vectors 0.80 to 0.98; 16, 32 and 48 1.05 to 1.37, 9 to 12 up to 1.29, 22 up to 1.19).  In FP64 (p = 7, 8) they leave:
//   12 vectors gained 10% at 1.2e6 nodes and lost up to 15% below, the other counts lose everywhere.
constexpr bool mline_serves(int P, int Q, int mode, bool colloc, int elem_bytes, int v, int nvec, int nex, int64_t nelem)
{
    if (!mline_variant(mode, colloc, v)) return false;
    const int vc = variant_vc(v), chunks = (nvec + vc - 1) / vc;
    const bool f32 = elem_bytes == 4;
    const int rows = v == 6                ? (nvec == 3 ? kMlineRows3 : kMlineRows4)[Q - 2]
                     : nvec > 14 && Q >= 4 ? (Q == 5 ? 2 : 1)
                                           : (f32 ? kMlineRows8f32 : kMlineRows8)[Q - 2];
    if (nex < rows) return false;
    if (chunks == 1 && (!cached_factors(Q, elem_bytes, nelem) || (f32 ? nvec != 4 : v != 7 || nvec < 8))) return true;
    if (vc * elem_bytes >= 64) return nvec > 12 || !cached_factors(Q, elem_bytes, nelem);
    if (chunks == 1) return false;
    if (nelem <= kFewElements) return true;
    if (f32) return Q == 2 || Q > 6 || (Q == 3 ? nvec % 16 != 0 : nvec % 16 == 8);
    return apply_lds(P, Q, mode, elem_bytes, v, true) > kLdsTwoGroups;
}

// Single-vector launch defaults of the line-fused kernel per q (index q-2).  Measured time of every
// slot in percent of the best, at about 1e7 nodes and with the idle elements of ragged x rows taken
// out; the default is the slot with the smallest time x idle share on the operator's own row length
// (a row of nex elements takes ceil(nex / G) groups of G).  At p = 5 (G = 5: 201 us for whole rows,
// G = 1: 242) a row of 6 elements is 17% faster with G = 1.
constexpr int kLineCostDiff[9][5] = {{100, 100, 130, 100, 250}, {103, 101, 100, 162, 306}, {108, 102, 100, 169, 310},
                                     {100, 101, 120, 117, 194}, {100, 111, 102, 132, 126}, {100, 121, 122, 109, 113},
                                     {106, 110, 100, 104, 109}, {100, 139, 114, 139, 100}, {107, 148, 100, 107, 100}};
constexpr int kLineCostColl[9][5] = {{102, 102, 137, 100, 245}, {100, 107, 105, 148, 259}, {100, 115, 116, 143, 232},
                                     {105, 100, 136, 115, 192}, {100, 111, 114, 188, 150}, {100, 162, 129, 115, 122},
                                     {108, 137, 113, 100, 137}, {117, 130, 100, 130, 117}, {107, 148, 100, 107, 100}};
constexpr int kLineCostMass[9][5] = {{107, 101, 100, 157, 277}, {107, 101, 100, 157, 277}, {114, 103, 100, 178, 308},
                                     {112, 100, 167, 124, 255}, {100, 126, 106, 198, 138}, {100, 175, 133, 105, 106},
                                     {120, 152, 100, 111, 152}, {100, 146, 113, 146, 100}, {129, 100, 101, 129, 101}};
// FP32 diffusion (p = 1..8, 1e7 nodes, Gauss: 1583 -> 1079, 384 -> 342, 287 -> 223, 213 -> 182, 193 -> 155, 168 -> 130,
// 165 -> 128, 169 -> 155 us against the stored-factor kernel): medians over boxes of 1e6 to 1e7 nodes.  An idle element
// counts 0.4 of a used one (its lanes skip the loads and atomics), which keeps the choice within 20% of the fastest slot
// for rows of 1 to 25 elements at 2e5 and 2e6 nodes; counted in full it was up to 39% off.  One slot for every row length
// took up to twice as long on short rows: collocated p = 2, rows of 1 .. 7 at 2e6 nodes 214 .. 64 us with groups of 14,
// 119 .. 43 with the row's own; Gauss p = 7, rows of one 64, 40.
constexpr int kIdle32Percent = 40;
constexpr int kLineCost32Diff[9][5] = {{103, 100, 102, 156, 276}, {103, 100, 102, 156, 276}, {117, 103, 100, 171, 323},
                                       {102, 100, 117, 118, 200}, {100, 108, 101, 147, 139}, {100, 132, 115, 110, 116},
                                       {111, 140, 100, 104, 140}, {100, 141, 115, 141, 100}, {113, 159, 100, 113, 100}};
constexpr int kLineCost32Coll[9][5] = {{106, 100, 130, 102, 223}, {102, 100, 100, 135, 226}, {113, 100, 112, 150, 258},
                                       {107, 100, 142, 116, 234}, {100, 114, 107, 220, 158}, {100, 183, 139, 113, 121},
                                       {127, 157, 100, 107, 157}, {100, 136, 107, 136, 100}, {113, 159, 100, 113, 100}};
// FP32 diffusion on meshes of at most kFewElements, which take a launch's time (12 us) in any slot.
constexpr int kLineSlot32Gauss[9] = {0, 0, 0, 0, 0, 0, 0, 0, 2};
constexpr int kLineSlot32Coll[9] = {0, 1, 0, 1, 0, 3, 2, 2, 2};
// One-vector collocated diffusion in FP64 where the stored-factor kernel (k_apply) is faster than k_line: rows of at most
// `rows` elements, which waste the lanes of its groups least, and meshes whose stored factors take at most mb MB, which the
// 256 MB Infinity Cache feeds.  us of k_apply and of k_line's best slot: p = 1, rows of 1, 4, 9, 13 at 2e6 nodes 509 572,
// 260 298, 180 187, 172 168, 66^3 elements (110 MB) 30 33, 99^3 (373 MB) 93 88, 214^3 948 747; p = 8, rows of one with a
// coefficient 42 45, without 40 40 (rows of two 48 35).
// FP32 launches evaluate their factors in FP64 everywhere, for half the error (1.6e-7 against 2.9e-7 at p = 3), also where
// factors stored in FP32 would be faster: collocated p = 1, 66^3 elements 32 us against 24, rows of 4 239 against 161; p = 3,
// rows of 4 36, 29; Gauss p = 2, 33^3 and 72^3 19, 118 against 15, 121; p = 7, rows of one 40, 31.
struct ElemRange {
    int rows, mb;
};
constexpr ElemRange kElemColl[9] = {{9, 256}, {}, {}, {}, {}, {}, {}, {1, 0}, {}};
// Mass, k_line: largest automatic pipeline depth (elements a group marches through).
constexpr int kDefChainLineMass[9] = {8, 8, 8, 8, 4, 2, 4, 4, 2};
// k_mass (collocated, and several vectors with Gauss points): the collocated one-vector variant, and the depth.  With
// k_line's depths several vectors of Gauss mass took up to 2.8 times as long (p = 2, 1e4 nodes of 12 vectors: 12 us, 33).
constexpr int kDefVariantMassColl[9] = {0, 0, 0, 3, 3, 1, 3, 0, 4};
constexpr int kDefChainMass[9] = {2, 2, 2, 4, 2, 4, 4, 4, 2};
// Device basis block (elements): B [Q][P], B^T [P][Q], D [Q][Q], D^T [Q][Q],
// then the folded (even-odd) forms of the same four matrices: for a matrix M
// with NO rows and NI columns, row o < ceil(NO/2) holds
//   [ (M[o][i] + M[o][NI-1-i])/2 for i < NI/2 | (M[o][i] - M[o][NI-1-i])/2 for i < NI/2 | M[o][NI/2] if NI odd ].
constexpr int half_up(int n) { return (n + 1) / 2; }
constexpr int basis_b(int, int) { return 0; }
constexpr int basis_bt(int P, int Q) { return Q * P; }
constexpr int basis_d(int P, int Q) { return 2 * Q * P; }
constexpr int basis_dt(int P, int Q) { return 2 * Q * P + Q * Q; }
constexpr int basis_bf(int P, int Q) { return 2 * Q * P + 2 * Q * Q; }
constexpr int basis_btf(int P, int Q) { return basis_bf(P, Q) + half_up(Q) * P; }
constexpr int basis_df(int P, int Q) { return basis_btf(P, Q) + half_up(P) * Q; }
constexpr int basis_dtf(int P, int Q) { return basis_df(P, Q) + half_up(Q) * Q; }
constexpr int basis_xq(int P, int Q) { return basis_dtf(P, Q) + half_up(Q) * Q; }  // quadrature points [Q]
constexpr int basis_wq(int P, int Q) { return basis_xq(P, Q) + Q; }                  // quadrature weights [Q]
// folded G [Q][P] (G[a][i] = l_i'(x_a), the basis derivative at the points); the block ends in half_up(P) * Q elements
// that nothing uses, which keep the workspace sizes that callers have been told
constexpr int basis_gf(int P, int Q) { return basis_wq(P, Q) + Q; }
constexpr int basis_len(int P, int Q) { return basis_gf(P, Q) + half_up(Q) * P + half_up(P) * Q; }

// Per-order dispatch (one translation unit per order, apply_p<N>.hip).
hipError_t launch_apply(const ApplyLaunch &a);
hipError_t launch_kgrad(const KgradLaunch &a);
hipError_t launch_diag(const DiagLaunch &a);

#define MFHEX_DECLARE_ORDER(N)                                  \
    hipError_t launch_apply_p##N(const ApplyLaunch &a);         \
    hipError_t launch_kgrad_p##N(const KgradLaunch &a);         \
    hipError_t launch_diag_p##N(const DiagLaunch &a);
MFHEX_DECLARE_ORDER(1)
MFHEX_DECLARE_ORDER(2)
MFHEX_DECLARE_ORDER(3)
MFHEX_DECLARE_ORDER(4)
MFHEX_DECLARE_ORDER(5)
MFHEX_DECLARE_ORDER(6)
MFHEX_DECLARE_ORDER(7)
MFHEX_DECLARE_ORDER(8)

// Setup kernels (setup.hip).
struct GeomLaunch {
    int32_t nex, ney, nez, p, q;
    const double *vert;      // device copy of the vertices
    const Basis1D *basis;
    hipStream_t stream;
};
// Quadrature data: diffusion -> 6 factors w adj(J) adj(J)^T / detJ per point,
// mass -> w detJ.  q32 (optional) gets the FP32 rounding, wdet (optional) w detJ.
// bad gets a nonzero value if some detJ <= 0 (caller zeroes it first).
hipError_t launch_qdata(const GeomLaunch &g, int kind, double *q64, float *q32, double *wdet, int32_t *bad);
// Deterministic transposed restriction: y[n][v] (+)= sum of the element values ebuf[e][local][v] of
// the (up to 8) elements holding node n, in increasing element order; masked nodes keep y (add) or
// get 0.  prec: MFHEX_F64 / MFHEX_F32.
hipError_t launch_det_assemble(const GeomLaunch &g, int dirichlet, int nvec, int prec, const void *ebuf, void *y,
                               bool add);
hipError_t launch_offsets(const GeomLaunch &g, int dirichlet, int32_t *off);
hipError_t launch_qpoint_coords(const GeomLaunch &g, double *xyz);
hipError_t launch_node_coords(const GeomLaunch &g, double *xyz);

}  // namespace mfhex
