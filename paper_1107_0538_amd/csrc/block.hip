// Block Jacobi-PCG for s <= 64 right-hand sides: O'Leary's block conjugate
// gradients (the paper's CG iteration, Section IV, on a block of vectors) in
// the breakdown-free form of Ji and Li, whose search blocks are
// orthonormalised with rank revelation by shifted Cholesky QR (Fukaya et al.).
//
// Per iteration, on N x 64 row-major FP64 blocks (columns >= s are zero):
//   Q = A P                                  k_bc_spmm (row products, four rows a wave)
//   Gamma = P'Q, Psi = P'R                   k_bc_gram<2> + k_bc_sum
//   alpha = Gamma^-1 Psi                     k_bc_alpha (Cholesky over the live
//                                            columns, inverse factor)
//   X += P alpha                             k_bc_gemm<XUP>
//   R -= Q alpha, ||r_j||^2                  k_bc_gemm<RUP>
//   Q'Z, Z = M^-1 R                          k_bc_gram<1> + k_bc_sum (the norms too)
//   test, beta = -Gamma^-1 Q'Z               k_bc_beta
//   W = Z + P beta, W'W                      k_bc_gemm<DIR> + k_bc_sum
//   three CholeskyQR passes of W -> P        (k_bc_orth, k_bc_gemm<APPLY> with the
//                                            next pass's Gram matrix, k_bc_sum) x 3
// The Gram and block-times-64x64 products are dense contractions: they run on
// the FP64 matrix cores (v_mfma_f64_16x16x4f64), operands straight from
// global memory into the fragment layout.  The 64 x 64 factorisations run in
// one workgroup, in blocks of 16 columns.  All kernels of an
// iteration are captured in hipGraph chunks and return at entry once the
// state is no longer RUN; the host confirms a
// passed recurrence test on the true residuals and restarts the block from
// them if a column fails.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <utility>

#include "spmm.hpp"

namespace jpcg {

constexpr int kB = 64;       // block width inside the solver
constexpr int kBB = kB * kB;
typedef double d4 __attribute__((ext_vector_type(4)));

enum BcStatus : int { BC_RUN = 0, BC_PENDING = 1, BC_CONVERGED = 2, BC_MAXIT = 3, BC_BREAKDOWN = 4 };

struct BcState {
    int status;
    int k;         // iterations completed
    int maxit;
    int s;         // caller's block width
    int n;
    int restarts;
    int rank;      // live columns of P
    int pad;
    int live[kB];  // column j of P belongs to the basis
    double tol;
    double tau;    // rank cut-off of the second and third CholeskyQR passes
    double nb[kB];
    double thr2[kB];
    double rr[kB];   // ||r_j||^2 of the recurrence (or of the true residual after a check)
    double G0[kBB];  // reduced Gram matrices
    double G1[kBB];
    double Li[kBB];  // inverse Cholesky factor of Gamma = P'Q over the live columns
    double M[kBB];   // the 64 x 64 matrix the next block pass applies
};

__device__ __forceinline__ bool bc_stopped(const BcState* st, int gate)
{
    return gate && __builtin_amdgcn_readfirstlane(st->status) != BC_RUN;
}

// ---------------------------------------------------------------------------
// Gram products C_o = U' V_o (64 x 64) of N x 64 blocks, one per operand o.
// Fragment layouts of v_mfma_f64_16x16x4f64 (D = A B, A 16 x 4, B 4 x 16):
// lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and D[l / 16 + 4 v][l % 16]
// in slot v.  For C = U'V the reduction index is the row: A[i][k] =
// U[r0 + k][16 ib + i], B[k][j] = V[r0 + k][16 jb + j], so lane l loads
// U[r0 + l / 16][16 ib + l % 16] -- four rows of 128 contiguous bytes per
// block of 16 columns.  Each wave accumulates all 16 output tiles of its
// operand over its rows; waves of a workgroup are added in LDS in wave order
// and each workgroup writes one partial per operand.
// NOP = 2: half the waves take V0 and half V1 (U is read twice, from L2).
// NOP = 1: V0's rows are scaled (Q'Z with Z = M^-1 R formed here).
// Bound by the loads in flight: 8 waves a CU with 8 KB each ahead; 51^3, three
// blocks (204 MB) 54 us against 69 with 4 waves and 4 KB, two 33 against 39.
// ---------------------------------------------------------------------------
constexpr int kGramBS = 512;
constexpr int kGramStep = 8;  // rows of a wave's step

template <int NOP>
__global__ __launch_bounds__(kGramBS, 2) void k_bc_gram(int n, const double* __restrict__ U,
                                                     const double* __restrict__ V0, const double* __restrict__ V1,
                                                     const double* __restrict__ scale, double* __restrict__ part,
                                                     int rows_per_wg, int G, const BcState* st, int gate)
{
    if (bc_stopped(st, gate)) return;
    __shared__ double red[NOP][kBB];
    const int L = xcd_logical_block((int)blockIdx.x, G);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    constexpr int kWavesPerOp = kGramBS / kWave / NOP;
    const int op = w / kWavesPerOp, sub = w % kWavesPerOp;
    const double* __restrict__ V = op == 0 ? V0 : V1;
    const int rs = min(L * rows_per_wg, n), re = min(rs + rows_per_wg, n);
    d4 acc[4][4];
#pragma unroll
    for (int ib = 0; ib < 4; ++ib)
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) acc[ib][jb] = d4{0.0, 0.0, 0.0, 0.0};
    const int rq = lane >> 4, cq = lane & 15;
    // The loads of the next step are issued before this step's products.
    constexpr int Q = kGramStep / 4;
    double a[Q][4], b[Q][4], d[Q];
    auto fetch = [&](int r0) {
#pragma unroll
        for (int h = 0; h < Q; ++h) {
            const int row = r0 + 4 * h + rq;
            const bool ok = row < re;
            const size_t o = (size_t)(ok ? row : rs) * kB + cq;
            d[h] = 1.0;
            if (NOP == 1) d[h] = scale[ok ? row : rs];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                a[h][q] = ok ? U[o + 16 * q] : 0.0;
                b[h][q] = ok ? V[o + 16 * q] : 0.0;
            }
        }
    };
    int r0 = rs + kGramStep * sub;
    if (r0 < re) fetch(r0);
    while (r0 < re) {
        double ca[Q][4], cb[Q][4];
#pragma unroll
        for (int h = 0; h < Q; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ca[h][q] = a[h][q];
                cb[h][q] = NOP == 1 ? d[h] * b[h][q] : b[h][q];
            }
        r0 += kGramStep * kWavesPerOp;
        if (r0 < re) fetch(r0);
#pragma unroll
        for (int h = 0; h < Q; ++h)
#pragma unroll
            for (int ib = 0; ib < 4; ++ib)
#pragma unroll
                for (int jb = 0; jb < 4; ++jb)
                    acc[ib][jb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ca[h][ib], cb[h][jb], acc[ib][jb], 0, 0, 0);
    }
    // Add the waves of each operand in wave order.
    for (int t = 0; t < kWavesPerOp; ++t) {
        if (sub == t) {
#pragma unroll
            for (int ib = 0; ib < 4; ++ib)
#pragma unroll
                for (int jb = 0; jb < 4; ++jb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int e = (16 * ib + rq + 4 * v) * kB + 16 * jb + cq;
                        const double x = acc[ib][jb][v];
                        red[op][e] = t == 0 ? x : red[op][e] + x;
                    }
        }
        __syncthreads();
    }
    double* out = part + (size_t)L * NOP * kBB;
    for (int e = threadIdx.x; e < NOP * kBB; e += kGramBS) out[e] = red[e / kBB][e % kBB];
}

// dst[e] = sum over g of part[g * count + e] for e < count, in a fixed order:
// a workgroup takes EPB consecutive entries; its 256 / EPB thread groups add
// the partials g = q, q + groups, ... (group q), and the group sums are added
// in group order.  Gram partials: entries [0, 4096) to st->G0 and [4096, 8192)
// to st->G1.  The workgroups past those, if any, add the column norms' partials
// (norms[g * 64 + j], g < Gn) to st->rr: a launch of their own costs 3 us an
// iteration.
constexpr int kSumEntries = 32;

__global__ __launch_bounds__(256) void k_bc_sum(const double* __restrict__ part, int G, int count,
                                                const double* __restrict__ norms, int Gn, BcState* st, int gate)
{
    if (bc_stopped(st, gate)) return;
    constexpr int EPB = kSumEntries, kGroups = 256 / EPB;
    __shared__ double red[kGroups][EPB];
    const int j = threadIdx.x % EPB, q = threadIdx.x / EPB;
    const bool norm = (int)blockIdx.x * EPB >= count;
    const int e = blockIdx.x * EPB + j - (norm ? count : 0);
    if (norm) {
        part = norms;
        G = Gn;
        count = kB;
    }
    double s = 0.0;
    {
        int g = q;
        for (; g + 3 * kGroups < G; g += 4 * kGroups) {
            const double a0 = part[(size_t)g * count + e], a1 = part[(size_t)(g + kGroups) * count + e];
            const double a2 = part[(size_t)(g + 2 * kGroups) * count + e], a3 = part[(size_t)(g + 3 * kGroups) * count + e];
            s += (a0 + a1) + (a2 + a3);
        }
        for (; g < G; g += kGroups) s += part[(size_t)g * count + e];
    }
    red[q][j] = s;
    __syncthreads();
    if (q == 0) {
        double t = 0.0;
        for (int k = 0; k < kGroups; ++k) t += red[k][j];
        if (norm) st->rr[e] = t;
        else (e < kBB ? st->G0[e] : st->G1[e - kBB]) = t;
    }
}

// ---------------------------------------------------------------------------
// Block times 64 x 64: U M with U N x 64 and M = st->M.  Per wave a tile of
// 16 rows: D (16 x 64) = sum over 16 steps t of A_t B_t with the reduction
// index permuted so that lane l's A values are 16 contiguous entries of one
// row: step t, lane l holds A = U[r0 + l % 16][16 (l / 16) + t] and
// B = M[16 (l / 16) + t][16 jb + l % 16] (read from LDS).
//   BC_XUP:   Y += U M                     (X += P alpha)
//   BC_RUP:   Y -= U M, per-column partials of y'y  (R -= Q alpha, ||r_j||^2)
//   BC_DIR:   Y = D Z + U M                (W = M^-1 R + P beta)
//   BC_SCALE: Y = D Z                      (W = M^-1 R, the first direction)
//   BC_APPLY: Y = U M
// GRAM: the workgroup's share of Y'Y too.  The tile's rows are in the lanes as
// the matrix instructions want both operands of a Gram step, so a 16-row tile
// costs 40 more of them (the upper triangle of 16 x 16 blocks) and no memory:
// at 51^3 46 us with the Gram matrix, where the product took 33 and a pass for
// the Gram matrix another 33 (136 and 68 MB).  R -= Q alpha without a stored Z and
// with R's loads ahead of the products: 39 us, 87 before; W with its Gram matrix
// 50, 66 + 33 before.
// ---------------------------------------------------------------------------
enum BcGemm : int { BC_XUP = 0, BC_RUP = 1, BC_DIR = 2, BC_APPLY = 3, BC_SCALE = 4 };
constexpr int kGemmBS = 512;
constexpr int kGemmWaves = kGemmBS / kWave;
constexpr int kMPad = 65;  // LDS row pitch of M (doubles)

struct BcGemmArgs {
    int n;
    const double* U;
    double* Y;
    const double* Z;     // BC_DIR, BC_SCALE
    const double* dinv;  // the same
    double* part;        // BC_RUP: [G][64] partials of y'y
    double* gram;        // GRAM: [G][64 * 64]
    int G;
};

__device__ __forceinline__ void bc_tile_load(const double* __restrict__ U, int r0, int n, double (&a)[16])
{
    const int lane = threadIdx.x & 63, rq = lane >> 4, cq = lane & 15;
    const int row = r0 + cq;
    const bool ok = row < n;
    const double2* src = (const double2*)(U + (size_t)(ok ? row : 0) * kB + 16 * rq);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const double2 v = ok ? src[t] : make_double2(0.0, 0.0);
        a[2 * t] = v.x;
        a[2 * t + 1] = v.y;
    }
}

__device__ __forceinline__ void bc_tile_product(const double (&a)[16], const double* Ms, d4 (&acc)[4])
{
    const int lane = threadIdx.x & 63, rq = lane >> 4, cq = lane & 15;
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) acc[jb] = d4{0.0, 0.0, 0.0, 0.0};
    // Four steps' entries of M at a time: read all at once they take 128 registers.
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        if (t % 4 == 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
            acc[jb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], Ms[(16 * rq + t) * kMPad + 16 * jb + cq], acc[jb], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
}

template <int MODE, bool GRAM>
__global__ __launch_bounds__(kGemmBS, 2) void k_bc_gemm(BcGemmArgs g, BcState* st, int gate)
{
    if (bc_stopped(st, gate)) return;
    __shared__ double Ms[kB * kMPad];
    __shared__ double red[GRAM ? kBB : kGemmWaves * kB];
    if (MODE != BC_SCALE) {
        for (int e = threadIdx.x; e < kBB; e += kGemmBS) Ms[(e / kB) * kMPad + e % kB] = st->M[e];
        __syncthreads();
    }
    const int L = xcd_logical_block((int)blockIdx.x, g.G);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, rq = lane >> 4, cq = lane & 15;
    const int tiles = (g.n + 15) / 16;
    const int tpw = (tiles + g.G - 1) / g.G;
    const int t0 = min(L * tpw, tiles), t1 = min(t0 + tpw, tiles);
    double nrm[4] = {0.0, 0.0, 0.0, 0.0};
    d4 gr[GRAM ? 10 : 1];  // blocks (ib, jb), ib <= jb
    if constexpr (GRAM) {
#pragma unroll
        for (int e = 0; e < 10; ++e) gr[e] = d4{0.0, 0.0, 0.0, 0.0};
    }
    if (MODE == BC_XUP && L == 0 && threadIdx.x == 0) st->k += 1;
    // The next tile's row loads are issued before this tile's products.
    double a[16];
    int tile = t0 + w;
    if (MODE != BC_SCALE && tile < t1) bc_tile_load(g.U, tile * 16, g.n, a);
    while (tile < t1) {
        const int r0 = tile * 16;
        double ca[16], y[4][4];
#pragma unroll
        for (int u = 0; u < 16; ++u) ca[u] = a[u];
        // The rows of Y or Z that the product is added to.
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = min(r0 + rq + 4 * v, g.n - 1);
            double di = 1.0;
            if constexpr (MODE == BC_DIR || MODE == BC_SCALE) di = g.dinv[row];
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) {
                const size_t o = (size_t)row * kB + 16 * jb + cq;
                if constexpr (MODE == BC_XUP || MODE == BC_RUP) y[jb][v] = g.Y[o];
                if constexpr (MODE == BC_DIR || MODE == BC_SCALE) y[jb][v] = di * g.Z[o];
            }
        }
        tile += kGemmWaves;
        if (MODE != BC_SCALE && tile < t1) bc_tile_load(g.U, tile * 16, g.n, a);
        d4 acc[4];
        if constexpr (MODE != BC_SCALE) bc_tile_product(ca, Ms, acc);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = r0 + rq + 4 * v;
            const bool ok = row < g.n;
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) {
                const size_t o = (size_t)row * kB + 16 * jb + cq;
                double x;
                if constexpr (MODE == BC_XUP || MODE == BC_DIR) x = y[jb][v] + acc[jb][v];
                else if constexpr (MODE == BC_RUP) x = y[jb][v] - acc[jb][v];
                else if constexpr (MODE == BC_SCALE) x = y[jb][v];
                else x = acc[jb][v];
                if (ok) g.Y[o] = x;
                else x = 0.0;
                if constexpr (MODE == BC_RUP) nrm[jb] += x * x;
                if constexpr (GRAM) y[jb][v] = x;
            }
            if constexpr (GRAM) {
                int e = 0;
#pragma unroll
                for (int ib = 0; ib < 4; ++ib)
#pragma unroll
                    for (int jb = ib; jb < 4; ++jb, ++e)
                        gr[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[ib][v], y[jb][v], gr[e], 0, 0, 0);
            }
        }
    }
    if constexpr (MODE == BC_RUP) {
        // Column 16 jb + cq: lanes cq, cq + 16, cq + 32, cq + 48, then the waves in order.
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            double x = nrm[jb];
            x += __shfl_xor(x, 16);
            x += __shfl_xor(x, 32);
            nrm[jb] = x;
        }
        if (rq == 0) {
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) red[w * kB + 16 * jb + cq] = nrm[jb];
        }
        __syncthreads();
        if (threadIdx.x < kB) {
            double x = 0.0;
            for (int t = 0; t < kGemmWaves; ++t) x += red[t * kB + threadIdx.x];
            g.part[(size_t)L * kB + threadIdx.x] = x;
        }
    }
    if constexpr (GRAM) {
        // The waves in order; the triangle below is the one above.
        for (int t = 0; t < kGemmWaves; ++t) {
            if (w == t) {
                int e = 0;
#pragma unroll
                for (int ib = 0; ib < 4; ++ib)
#pragma unroll
                    for (int jb = ib; jb < 4; ++jb, ++e)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            double& o = red[(16 * ib + rq + 4 * v) * kB + 16 * jb + cq];
                            o = t == 0 ? gr[e][v] : o + gr[e][v];
                        }
            }
            __syncthreads();
        }
        double* out = g.gram + (size_t)L * kBB;
        for (int e = threadIdx.x; e < kBB; e += kGemmBS) {
            const int i = e / kB, j = e % kB;
            out[e] = i / 16 <= j / 16 ? red[e] : red[j * kB + i];
        }
    }
}

// ---------------------------------------------------------------------------
// Row products and residuals.
// ---------------------------------------------------------------------------

// Y = A X over N x 64 blocks (spmm.hpp).
template <SpmmKind KIND>
__global__ __launch_bounds__(kSpmmBS, spmm_waves(KIND)) void k_bc_spmm(RunMap<double> m, const double* __restrict__ X,
                                                     double* __restrict__ Y, int G, const BcState* st, int gate)
{
    if (bc_stopped(st, gate)) return;
    spmm_block<KIND>(m, X, Y, kB, G);
}

// R = B - AX (AX given), per-workgroup partials of r'r and b'b
// (part[g][0][64], part[g][1][64]); write = 0 only measures.
__global__ __launch_bounds__(256) void k_bc_residual(int n, const double* __restrict__ B,
                                                     const double* __restrict__ AX, double* __restrict__ R,
                                                     double* __restrict__ part, int write)
{
    __shared__ double red[2][4][kB];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double rr = 0.0, bb = 0.0;
    for (int i = blockIdx.x * 4 + w; i < n; i += gridDim.x * 4) {
        const size_t o = (size_t)i * kB + lane;
        const double b = B[o], r = b - AX[o];
        if (write) R[o] = r;
        rr += r * r;
        bb += b * b;
    }
    red[0][w][lane] = rr;
    red[1][w][lane] = bb;
    __syncthreads();
    if (threadIdx.x < kB) {
        const int j = threadIdx.x;
        part[((size_t)blockIdx.x * 2 + 0) * kB + j] = ((red[0][0][j] + red[0][1][j]) + red[0][2][j]) + red[0][3][j];
        part[((size_t)blockIdx.x * 2 + 1) * kB + j] = ((red[1][0][j] + red[1][1][j]) + red[1][2][j]) + red[1][3][j];
    }
}

// Copy between the caller's n x s block (leading dimension s) and the
// solver's n x 64 block (columns >= s zero).
__global__ void k_bc_pack(int n, int s, const double* __restrict__ src, double* __restrict__ dst, int to_wide)
{
    const int lane = threadIdx.x & 63;
    for (int i = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64; i < n; i += gridDim.x * (blockDim.x / 64)) {
        if (to_wide) dst[(size_t)i * kB + lane] = lane < s ? src[(size_t)i * s + lane] : 0.0;
        else if (lane < s) dst[(size_t)i * s + lane] = src[(size_t)i * kB + lane];
    }
}

// ---------------------------------------------------------------------------
// 64 x 64 factorisations, one workgroup of four waves, matrices in LDS.
//
// What bounds them is the chain of 64 pivots.  One wave with a column of the
// matrix per lane took 52 us for a Cholesky factor and its inverse, about 400 ns
// a step: a square root, a division, and the factor's column through LDS to 63
// updates.  In blocks of 16 columns a step updates the block's later columns
// only, from v_readlane broadcasts, with a reciprocal square root in place of
// root and division; what is left and the blocks of the inverse are products
// for the matrix cores: 21 us (31 with branches in the steps and with loads that
// each waited to be stored).
// ---------------------------------------------------------------------------
constexpr int kSmallBS = 256;
constexpr int kSP = 65;  // LDS pitch
constexpr int kBlk = 16;

// 1 / sqrt(d) for a normal d > 0: the hardware's estimate and two
// third-order Newton steps (the second one rounds).
__device__ __forceinline__ double recip_sqrt(double d)
{
    double x = __builtin_amdgcn_rsq(d);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const double e = __builtin_fma(-d * x, x, 1.0);
        x = __builtin_fma(x * e, __builtin_fma(0.375, e, 0.5), x);
    }
    return x;
}

// Fragments of the 16 x 16 x 4 FP64 product: a block's step t as left or right
// operand, and where slot v of a product lies.
struct Frag {
    int r, c;  // lane / 16, lane % 16
    __device__ Frag() : r((threadIdx.x & 63) >> 4), c(threadIdx.x & 15) {}
    // S[row0 + c][col0 + 4 t + r]: left operand, or right operand of the transpose.
    __device__ double rows(const double* S, int row0, int col0, int t) const
    {
        return S[(row0 + c) * kSP + col0 + 4 * t + r];
    }
    // S[row0 + 4 t + r][col0 + c]: right operand, or left operand of the transpose.
    __device__ double cols(const double* S, int row0, int col0, int t) const
    {
        return S[(row0 + 4 * t + r) * kSP + col0 + c];
    }
};
__device__ __forceinline__ d4 mfma4(double a, double b, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// The columns 16 b ... of the trailing matrix, factored by one wave with a row
// per lane.  keep[k] is set for the factored ones, ip[k] to the inverse of the
// factor's diagonal (0 where not).
__device__ __forceinline__ void chol_panel(double* A, int b, unsigned long long usem, int mode, double tau, int* keep,
                                           double* ip, bool& bad)
{
    const int i = threadIdx.x, c0 = kBlk * b;
    double p[kBlk], mine = 0.0;
#pragma unroll
    for (int j = 0; j < kBlk; ++j) p[j] = i >= c0 ? A[i * kSP + c0 + j] : 0.0;
    const unsigned used = (unsigned)(usem >> c0) & 0xffffu;
    unsigned kept = 0;
    // Straight through: a branch costs more than what it would leave out.
#pragma unroll
    for (int k = 0; k < kBlk; ++k) {
        const double d = read_lane(p[k], c0 + k);
        const bool u = (used >> k) & 1u;
        const bool kk = u & (mode == 0 ? (d > 0.0) & (d < __builtin_huge_val()) : d > tau);
        bad |= mode == 0 && u && !kk;
        kept |= (unsigned)kk << k;
        const double inv = kk ? recip_sqrt(kk ? d : 1.0) : 0.0;
        mine = i == c0 + k ? inv : mine;
        const double l = kk & (i >= c0 + k) ? p[k] * inv : 0.0;
        p[k] = l;
#pragma unroll
        for (int j = k + 1; j < kBlk; ++j) p[j] = __builtin_fma(-l, read_lane(l, c0 + j), p[j]);
    }
    if (i >= c0 && i < c0 + kBlk) {
        keep[i] = (kept >> (i - c0)) & 1u;
        ip[i] = mine;
    }
#pragma unroll
    for (int j = 0; j < kBlk; ++j)
        if (i >= c0) A[i * kSP + c0 + j] = p[j];
}

// X = L^-1 for the Cholesky factor L of the symmetric matrix in A (lower
// triangle; overwritten), taking columns in order and restricted to the kept
// ones (rows and columns not kept are zero in X).  mode 0: every column in `use`
// must have a positive pivot (bad = 1 otherwise); mode 1: a column whose pivot
// is <= tau is dropped.  Called by the whole workgroup.
__device__ __forceinline__ void small_inverse_factor(double* A, const int* use, int mode, double tau, int* keep,
                                                     double* ip, int* bad, double* X)
{
    constexpr int NB = kB / kBlk;
    const int w = threadIdx.x / kWave;
    const Frag f;
    unsigned long long usem = 0;
    if (w == 0) usem = __ballot(use[threadIdx.x] != 0);
    bool badk = false;
    for (int b = 0; b < NB; ++b) {
        if (w == 0) chol_panel(A, b, usem, mode, tau, keep, ip, badk);
        __syncthreads();
        // The trailing blocks' lower triangle, a wave per block.
        int e = 0;
        for (int ib = b + 1; ib < NB; ++ib)
            for (int jb = b + 1; jb <= ib; ++jb, ++e) {
                if (e % NB != w) continue;
                d4 acc;
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] = A[(kBlk * ib + f.r + 4 * v) * kSP + kBlk * jb + f.c];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc = mfma4(-f.rows(A, kBlk * ib, kBlk * b, t), f.rows(A, kBlk * jb, kBlk * b, t), acc);
#pragma unroll
                for (int v = 0; v < 4; ++v) A[(kBlk * ib + f.r + 4 * v) * kSP + kBlk * jb + f.c] = acc[v];
            }
        __syncthreads();
    }
    if (threadIdx.x == 0 && badk) *bad = 1;
    // The diagonal blocks of the inverse, a wave per block, a column per lane.
    {
        const int c0 = kBlk * w, j = f.c;
        double x[kBlk];
#pragma unroll
        for (int i = 0; i < kBlk; ++i) x[i] = i == j ? 1.0 : 0.0;
#pragma unroll
        for (int m = 0; m < kBlk; ++m) {
            const double xm = x[m] * ip[c0 + m];
            x[m] = xm;
#pragma unroll
            for (int i = m + 1; i < kBlk; ++i) x[i] = __builtin_fma(-A[(c0 + i) * kSP + c0 + m], xm, x[i]);
        }
        if (f.r == 0) {
#pragma unroll
            for (int i = 0; i < kBlk; ++i) X[(c0 + i) * kSP + c0 + j] = keep[c0 + j] ? x[i] : 0.0;
        }
        for (int jb = w + 1; jb < NB; ++jb)
#pragma unroll
            for (int v = 0; v < 4; ++v) X[(c0 + f.r + 4 * v) * kSP + kBlk * jb + f.c] = 0.0;
    }
    __syncthreads();
    // Then the diagonals below: X_ij = -X_ii sum over k of L_ik X_kj.  The sum's
    // slots are the second product's right operands as they are.
    for (int d = 1; d < NB; ++d) {
        const int ib = w + d, jb = w;
        if (ib < NB) {
            d4 sum = {0.0, 0.0, 0.0, 0.0}, x = {0.0, 0.0, 0.0, 0.0};
            for (int kb = jb; kb < ib; ++kb)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    sum = mfma4(f.rows(A, kBlk * ib, kBlk * kb, t), f.cols(X, kBlk * kb, kBlk * jb, t), sum);
#pragma unroll
            for (int t = 0; t < 4; ++t) x = mfma4(-f.rows(X, kBlk * ib, kBlk * ib, t), sum[t], x);
#pragma unroll
            for (int v = 0; v < 4; ++v) X[(kBlk * ib + f.r + 4 * v) * kSP + kBlk * jb + f.c] = x[v];
        }
        __syncthreads();
    }
}

// op(A) B for 64 x 64 LDS matrices (op = transpose if ta): a wave takes 16 rows.
__device__ __forceinline__ void small_matmul(const double* A, int ta, const double* B, d4 (&c)[4])
{
    const int w = threadIdx.x / kWave;
    const Frag f;
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) c[jb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int t = 0; t < kB / 4; ++t) {
        const double a = ta ? f.cols(A, 0, kBlk * w, t) : f.rows(A, kBlk * w, 0, t);
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) c[jb] = mfma4(a, f.cols(B, 0, kBlk * jb, t), c[jb]);
    }
}

// The product to out[e] (global, row-major) scaled by `sign`.  Returns whether
// every entry (of the whole matrix) is finite.
__device__ __forceinline__ bool small_matmul_out(const double* A, int ta, const double* B, double sign, double* out)
{
    const int w = threadIdx.x / kWave;
    const Frag f;
    d4 c[4];
    small_matmul(A, ta, B, c);
    bool finite = true;
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            out[(kBlk * w + f.r + 4 * v) * kB + kBlk * jb + f.c] = sign * c[jb][v];
            finite = finite && isfinite(c[jb][v]);
        }
    return __syncthreads_and(finite ? 1 : 0) != 0;
}

// The product into an LDS matrix.
__device__ __forceinline__ void small_matmul_lds(const double* A, int ta, const double* B, double* C)
{
    const int w = threadIdx.x / kWave;
    const Frag f;
    d4 c[4];
    small_matmul(A, ta, B, c);
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int v = 0; v < 4; ++v) C[(kBlk * w + f.r + 4 * v) * kSP + kBlk * jb + f.c] = c[jb][v];
    __syncthreads();
}

__device__ void load_small(const double* src, double* dst)
{
    double v[kBB / kSmallBS];  // all loads in flight together
#pragma unroll
    for (int u = 0; u < kBB / kSmallBS; ++u) v[u] = src[threadIdx.x + u * kSmallBS];
#pragma unroll
    for (int u = 0; u < kBB / kSmallBS; ++u) {
        const int e = threadIdx.x + u * kSmallBS;
        dst[(e / kB) * kSP + e % kB] = v[u];
    }
    __syncthreads();
}

// alpha = Gamma^-1 Psi over the live columns (Gamma = G0 = P'Q, Psi = G1 = P'R):
// Cholesky of Gamma, Li = L^-1 kept for beta, M = Li' (Li Psi).
__global__ __launch_bounds__(kSmallBS) void k_bc_alpha(BcState* st, int gate)
{
    if (bc_stopped(st, gate)) return;
    __shared__ double A[kB * kSP], X[kB * kSP], T[kB * kSP], ip[kB];
    __shared__ int use[kB], keep[kB], bad;
    if (threadIdx.x == 0) bad = 0;
    if (threadIdx.x < kB) use[threadIdx.x] = st->live[threadIdx.x];
    load_small(st->G0, A);
    small_inverse_factor(A, use, 0, 0.0, keep, ip, &bad, X);
    if (bad) {
        if (threadIdx.x == 0) st->status = BC_BREAKDOWN;
        return;
    }
    for (int e = threadIdx.x; e < kBB; e += kSmallBS) st->Li[e] = X[(e / kB) * kSP + e % kB];
    load_small(st->G1, A);
    small_matmul_lds(X, 0, A, T);                             // T = Li Psi
    const bool finite = small_matmul_out(X, 1, T, 1.0, st->M);  // M = Li' T
    if (!finite && threadIdx.x == 0) st->status = BC_BREAKDOWN;
}

// Apply the stopping tests to the column norms of the updated residual
// (st->rr) and, if the iteration continues, M = beta = -Li' (Li Q'Z) (G0 = Q'Z).
__global__ __launch_bounds__(kSmallBS) void k_bc_beta(BcState* st, int gate)
{
    if (bc_stopped(st, gate)) return;
    __shared__ double A[kB * kSP], X[kB * kSP], T[kB * kSP];
    __shared__ int decide;
    const int t = threadIdx.x;
    if (t < kB) {
        // Lane j tests column j; the ballots give every lane the verdicts.
        const double rj = st->rr[t];
        const bool pass = __ballot(rj <= st->thr2[t]) == ~0ull;
        const bool finite = __ballot(isfinite(rj)) == ~0ull;
        int s = BC_RUN;
        if (!finite) s = BC_BREAKDOWN;
        else if (pass) s = BC_PENDING;
        else if (st->k >= st->maxit) s = BC_MAXIT;
        if (t == 0) {
            st->status = s;
            decide = s;
        }
    }
    __syncthreads();
    if (decide != BC_RUN) return;
    load_small(st->Li, X);
    load_small(st->G0, A);
    small_matmul_lds(X, 0, A, T);
    const bool finite = small_matmul_out(X, 1, T, -1.0, st->M);
    if (!finite && threadIdx.x == 0) st->status = BC_BREAKDOWN;
}

// One CholeskyQR pass on the Gram matrix G0 of the current block W:
// pass 0: columns scaled to unit norm, shift 11 (n s + s (s + 1)) u trace,
// no dropping; passes 1 and 2: columns dropped at a pivot <= tau.  M = the
// inverse transposed factor (times the scaling in pass 0); after pass 2 the
// kept columns are the live columns of the new P.
__global__ __launch_bounds__(kSmallBS) void k_bc_orth(BcState* st, int pass, int gate)
{
    if (bc_stopped(st, gate)) return;
    __shared__ double A[kB * kSP], X[kB * kSP], scale[kB], ip[kB];
    __shared__ int use[kB], keep[kB], bad;
    const int t = threadIdx.x;
    load_small(st->G0, A);
    if (t < kB) {
        const double d = A[t * kSP + t];
        scale[t] = pass == 0 ? (d > 0.0 ? 1.0 / sqrt(d) : 0.0) : 1.0;
        use[t] = 1;
    }
    if (t == 0) bad = 0;
    __syncthreads();
    if (pass == 0) {
        for (int e = t; e < kBB; e += kSmallBS) {
            const int i = e / kB, j = e % kB;
            A[i * kSP + j] *= scale[i] * scale[j];
        }
        __syncthreads();
        if (t < kB) {
            double tr = A[t * kSP + t];
            for (int off = kB / 2; off > 0; off /= 2) tr += __shfl_xor(tr, off);
            const double s = (double)st->s, n = (double)st->n;
            A[t * kSP + t] += 11.0 * (n * s + s * (s + 1.0)) * 0x1p-53 * tr;
        }
        __syncthreads();
    }
    small_inverse_factor(A, use, 1, pass == 0 ? 0.0 : st->tau, keep, ip, &bad, X);
    // M[i][j] = scale_i X[j][i]
    for (int e = t; e < kBB; e += kSmallBS) {
        const int i = e / kB, j = e % kB;
        st->M[e] = scale[i] * X[j * kSP + i];
    }
    if (pass == 2 && t < kB) {
        st->live[t] = keep[t];
        if (t == 0) {
            int r = 0;
            for (int j = 0; j < kB; ++j) r += keep[j];
            st->rank = r;
            if (r == 0) st->status = BC_BREAKDOWN;
        }
    }
}

// Set-up / check scalars from the residual partials (part[g][2][64]):
// mode 0 (set-up): nb, thresholds; status CONVERGED if every column passes,
// BREAKDOWN on a non-finite value, else RUN.  mode 1 (check of a PENDING
// state): CONVERGED if every true residual passes, else RUN and one more
// restart.  mode 2 (report): rr = ||b - A x||^2 only.
__global__ __launch_bounds__(1024) void k_bc_scalars(BcState* st, const double* __restrict__ part, int G, int mode)
{
    __shared__ double rr[kB], bb[kB], sums[16][2][kB];
    const int t = threadIdx.x;
    {
        // A wave takes every 16th workgroup's partials; the waves' sums in order.
        double a = 0.0, b = 0.0;
        const int j = t % kB, w = t / kB;
        for (int g = w; g < G; g += 16) {
            a += part[((size_t)g * 2 + 0) * kB + j];
            b += part[((size_t)g * 2 + 1) * kB + j];
        }
        sums[w][0][j] = a;
        sums[w][1][j] = b;
        __syncthreads();
    }
    if (t < kB) {
        double a = 0.0, b = 0.0;
        for (int w = 0; w < 16; ++w) {
            a += sums[w][0][t];
            b += sums[w][1][t];
        }
        rr[t] = a;
        bb[t] = b;
        st->rr[t] = a;
        if (mode == 0) {
            const double nb = sqrt(b);
            st->nb[t] = nb;
            const double thr = st->tol * nb;
            st->thr2[t] = thr * thr;
        }
    }
    __syncthreads();
    if (t == 0 && mode != 2) {
        bool pass = true, finite = true;
        for (int j = 0; j < kB; ++j) {
            pass = pass && rr[j] <= st->thr2[j];
            finite = finite && isfinite(rr[j]) && isfinite(bb[j]);
        }
        if (mode == 0) {
            st->k = 0;
            st->restarts = 0;
            for (int j = 0; j < kB; ++j) st->live[j] = 1;
        }
        if (!finite) st->status = BC_BREAKDOWN;
        else if (pass) st->status = BC_CONVERGED;
        else {
            if (mode == 1) st->restarts += 1;
            st->status = BC_RUN;
        }
    }
}

}  // namespace jpcg

// Block solver state hanging off a context.
struct cg_block {
    int gram_G = 0, gemm_G = 0, spmm_G = 0, gram_rpw = 0, res_G = 0, chunk = 4;
    double* work = nullptr;  // B, X, R, Z, P, Q, W: 7 n x 64 blocks
    double* part = nullptr;  // Gram partials [gram_G][2][4096], [gemm_G][4096]
    double* part2 = nullptr; // norm / residual partials [max(gemm_G, res_G)][2][64]
    jpcg::BcState* st = nullptr;
    jpcg::BcState* hst = nullptr;
    hipGraphExec_t exec = nullptr;
    double tol = -1.0, tau = -1.0;
    int maxit = -1;
};

namespace jpcg {

struct BcBufs {
    double *B, *X, *R, *Z, *P, *Q, *W;
};

static BcBufs bufs(cg_ctx* c, cg_block* b)
{
    const size_t nb = (size_t)c->n * kB;
    double* w = b->work;
    return {w, w + nb, w + 2 * nb, w + 3 * nb, w + 4 * nb, w + 5 * nb, w + 6 * nb};
}

void free_block(cg_ctx* c)
{
    cg_block* b = c->block;
    if (!b) return;
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->work) (void)hipFree(b->work);
    if (b->part) (void)hipFree(b->part);
    if (b->part2) (void)hipFree(b->part2);
    if (b->st) (void)hipFree(b->st);
    if (b->hst) (void)hipHostFree(b->hst);
    delete b;
    c->block = nullptr;
}

static void launch(const void* fn, int grid, int bs, hipStream_t st, void** args)
{
    JPCG_HIP(hipLaunchKernel(fn, dim3(grid), dim3(bs), args, 0, st));
}

// The kernels of the block operations, enqueued on `st`.
struct BcOps {
    cg_ctx* c;
    cg_block* b;
    BcBufs v;
    hipStream_t st;

    void spmm(const double* X, double* Y, int gate)
    {
        RunMap<double> m = run_map(c);
        void* a[] = {&m, &X, &Y, &b->spmm_G, &b->st, &gate};
        launch(c->streams ? (const void*)k_bc_spmm<SPMM_FOURS_STREAMS> : (const void*)k_bc_spmm<SPMM_FOURS>, b->spmm_G, kSpmmBS, st, a);
    }
    // With `norms` the column norms of the last BC_RUP too.
    void sum_grams(int nop, int G, int gate, bool norms = false)
    {
        int count = nop * kBB;
        void* r[] = {&b->part, &G, &count, &b->part2, &b->gemm_G, &b->st, &gate};
        launch((const void*)k_bc_sum, (count + (norms ? kB : 0)) / kSumEntries, 256, st, r);
    }
    void gram(const double* U, const double* V0, const double* V1, int gate, bool norms = false)
    {
        int n = c->n;
        const int nop = V1 ? 2 : 1;
        void* a[] = {&n, &U, &V0, &V1, &c->dinv, &b->part, &b->gram_rpw, &b->gram_G, &b->st, &gate};
        launch(nop == 2 ? (const void*)k_bc_gram<2> : (const void*)k_bc_gram<1>, b->gram_G, kGramBS, st, a);
        sum_grams(nop, b->gram_G, gate, norms);
    }
    // With `grams` also Y'Y.
    void gemm(int mode, const double* U, double* Y, const double* Z, int gate, bool grams = false)
    {
        BcGemmArgs g{c->n, U, Y, Z, c->dinv, b->part2, b->part, b->gemm_G};
        void* a[] = {&g, &b->st, &gate};
        const void* fn = mode == BC_XUP     ? (const void*)k_bc_gemm<BC_XUP, false>
                         : mode == BC_RUP   ? (const void*)k_bc_gemm<BC_RUP, false>
                         : mode == BC_DIR   ? (const void*)k_bc_gemm<BC_DIR, true>
                         : mode == BC_SCALE ? (const void*)k_bc_gemm<BC_SCALE, true>
                         : grams            ? (const void*)k_bc_gemm<BC_APPLY, true>
                                            : (const void*)k_bc_gemm<BC_APPLY, false>;
        launch(fn, b->gemm_G, kGemmBS, st, a);
        if (grams) sum_grams(1, b->gemm_G, gate);
    }
    void orth_pass(int pass, int gate)
    {
        void* a[] = {&b->st, &pass, &gate};
        launch((const void*)k_bc_orth, 1, kSmallBS, st, a);
    }
    // P = orth(W0): three CholeskyQR passes, the blocks in W0 -> Wa -> Wb -> P;
    // W0's Gram matrix is there.
    void orth(const double* W0, double* Wa, double* Wb, int gate)
    {
        orth_pass(0, gate);
        gemm(BC_APPLY, W0, Wa, nullptr, gate, true);
        orth_pass(1, gate);
        gemm(BC_APPLY, Wa, Wb, nullptr, gate, true);
        orth_pass(2, gate);
        gemm(BC_APPLY, Wb, v.P, nullptr, gate);
    }
    // P = orth(M^-1 R): the first direction.
    void start()
    {
        gemm(BC_SCALE, nullptr, v.W, v.R, 0, true);
        orth(v.W, v.Z, v.Q, 0);
    }
    // R = B - A X (write), partials of r'r, b'b; then the scalars.
    void residual(int write, int mode)
    {
        spmm(v.X, v.Q, 0);
        int n = c->n;
        void* a[] = {&n, &v.B, &v.Q, &v.R, &b->part2, &write};
        launch((const void*)k_bc_residual, b->res_G, 256, st, a);
        void* s[] = {&b->st, &b->part2, &b->res_G, &mode};
        launch((const void*)k_bc_scalars, 1, 1024, st, s);
    }
    // One gated iteration.
    void iteration()
    {
        spmm(v.P, v.Q, 1);
        gram(v.P, v.Q, v.R, 1);
        int gate = 1;
        void* a[] = {&b->st, &gate};
        launch((const void*)k_bc_alpha, 1, kSmallBS, st, a);
        gemm(BC_XUP, v.P, v.X, nullptr, 1);
        gemm(BC_RUP, v.Q, v.R, nullptr, 1);
        gram(v.Q, v.R, nullptr, 1, true);
        void* bta[] = {&b->st, &gate};
        launch((const void*)k_bc_beta, 1, kSmallBS, st, bta);
        gemm(BC_DIR, v.P, v.W, v.R, 1, true);
        // W -> Z -> Q -> P (Z and Q are free until the next iteration's product)
        orth(v.W, v.Z, v.Q, 1);
    }
};

static cg_block* make_block(cg_ctx* c)
{
    cg_block* b = new cg_block();
    try {
        const size_t nb = (size_t)c->n * kB;
        b->gram_G = std::max(8, std::min(c->cus, (c->n + 63) / 64) / 8 * 8);
        b->gram_rpw = (c->n + b->gram_G - 1) / b->gram_G;
        const int tiles = (c->n + 15) / 16;
        b->gemm_G = std::max(8, std::min(c->cus, (tiles + kGemmWaves - 1) / kGemmWaves) / 8 * 8);
        b->spmm_G = spmm_grid(c, spmm_blocks_per_cu(c));
        b->res_G = std::min(1024, (c->n + 3) / 4);
        JPCG_HIP(hipMalloc(&b->work, sizeof(double) * nb * 7));
        JPCG_HIP(hipMalloc(&b->part, sizeof(double) * (size_t)std::max(2 * b->gram_G, b->gemm_G) * kBB));
        JPCG_HIP(hipMalloc(&b->part2, sizeof(double) * (size_t)std::max(b->gemm_G, b->res_G) * 2 * kB));
        JPCG_HIP(hipMalloc(&b->st, sizeof(BcState)));
        JPCG_HIP(hipHostMalloc(&b->hst, sizeof(BcState), hipHostMallocDefault));
        JPCG_HIP(hipMemsetAsync(b->work, 0, sizeof(double) * nb * 7, c->stream));
        JPCG_HIP(hipMemsetAsync(b->st, 0, sizeof(BcState), c->stream));
        JPCG_HIP(hipStreamSynchronize(c->stream));
        return b;
    } catch (...) {
        if (b->work) (void)hipFree(b->work);
        if (b->part) (void)hipFree(b->part);
        if (b->part2) (void)hipFree(b->part2);
        if (b->st) (void)hipFree(b->st);
        if (b->hst) (void)hipHostFree(b->hst);
        delete b;
        throw;
    }
}

static void capture_block(cg_ctx* c, cg_block* b)
{
    if (b->exec) {
        (void)hipGraphExecDestroy(b->exec);
        b->exec = nullptr;
    }
    hipStream_t cap;
    JPCG_HIP(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
    BcOps ops{c, b, bufs(c, b), cap};
    hipGraph_t graph;
    JPCG_HIP(hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal));
    for (int it = 0; it < b->chunk; ++it) ops.iteration();
    JPCG_HIP(hipStreamEndCapture(cap, &graph));
    hipError_t e = hipGraphInstantiate(&b->exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    JPCG_HIP(e);
    JPCG_HIP(hipStreamDestroy(cap));
}

static BcState bc_read(cg_ctx* c, cg_block* b)
{
    JPCG_HIP(hipMemcpyAsync(b->hst, b->st, sizeof(BcState), hipMemcpyDeviceToHost, c->stream));
    JPCG_HIP(hipStreamSynchronize(c->stream));
    return *b->hst;
}

static void bc_set_status(cg_ctx* c, cg_block* b, int status)
{
    b->hst->status = status;
    JPCG_HIP(hipMemcpyAsync(b->st, b->hst, sizeof(int), hipMemcpyHostToDevice, c->stream));
}

}  // namespace jpcg

using namespace jpcg;

extern "C" {

int cg_solve_block(cg_ctx* c, const double* B, double* X, int32_t s, double tol, int32_t maxit, cg_info* info)
{
    if (!c) return CG_EINVAL;
    if (!B || !X || B == X || s < 1 || s > kB || !(tol >= 0.0) || !std::isfinite(tol))
        return set_error(c, CG_EINVAL, "cg_solve_block: bad arguments");
    if (maxit <= 0) maxit = c->n;
    try {
        if (!c->block) c->block = make_block(c);
        cg_block* b = c->block;
        hipStream_t st = c->stream;
        BcOps ops{c, b, bufs(c, b), st};
        // Parameters live in the state block; the graphs read them there.
        JPCG_HIP(hipStreamSynchronize(st));
        b->hst->tol = tol;
        b->hst->tau = 1e-14;
        b->hst->maxit = maxit;
        b->hst->s = s;
        b->hst->n = c->n;
        JPCG_HIP(hipMemcpyAsync(&b->st->tol, &b->hst->tol, sizeof(double) * 2, hipMemcpyHostToDevice, st));
        JPCG_HIP(hipMemcpyAsync(&b->st->maxit, &b->hst->maxit, sizeof(int) * 3, hipMemcpyHostToDevice, st));
        if (!b->exec) capture_block(c, b);
        JPCG_HIP(hipEventRecord(c->ev0, st));
        int n = c->n, one = 1, zero = 0;
        const int pg = std::min(4096, (c->n + 3) / 4);
        void* pb[] = {&n, &s, &B, &ops.v.B, &one};
        launch((const void*)k_bc_pack, pg, 256, st, pb);
        void* px[] = {&n, &s, &X, &ops.v.X, &one};
        launch((const void*)k_bc_pack, pg, 256, st, px);
        ops.residual(1, 0);
        BcState h = bc_read(c, b);
        if (h.status == BC_RUN) {
            ops.start();
            const long long guard = 2LL * maxit + 64;
            long long launched = 0;
            while (true) {
                JPCG_HIP(hipGraphLaunch(b->exec, st));
                JPCG_HIP(hipGraphLaunch(b->exec, st));
                launched += 2 * b->chunk;
                h = bc_read(c, b);
                if (h.status == BC_PENDING) {
                    // Confirm on the true residuals; restart from them if a column fails.
                    ops.residual(1, 1);
                    h = bc_read(c, b);
                    if (h.status == BC_RUN) {
                        if (h.k >= maxit) {
                            bc_set_status(c, b, BC_MAXIT);
                            h.status = BC_MAXIT;
                        } else {
                            for (int j = 0; j < kB; ++j) b->hst->live[j] = 1;
                            JPCG_HIP(hipMemcpyAsync(b->st->live, b->hst->live, sizeof(int) * kB, hipMemcpyHostToDevice, st));
                            ops.start();
                        }
                    }
                }
                if (h.status != BC_RUN) break;
                if (launched > guard) throw HipError{hipErrorUnknown, "block solver did not stop"};
            }
        }
        // True residual of the returned X for every column.
        ops.residual(0, 2);
        void* ux[] = {&n, &s, &ops.v.X, &X, &zero};
        launch((const void*)k_bc_pack, pg, 256, st, ux);
        JPCG_HIP(hipEventRecord(c->ev1, st));
        JPCG_HIP(hipEventSynchronize(c->ev1));
        const BcState f = bc_read(c, b);
        float ms = 0.f;
        JPCG_HIP(hipEventElapsedTime(&ms, c->ev0, c->ev1));
        const int code = h.status == BC_CONVERGED ? CG_CONVERGED : h.status == BC_MAXIT ? CG_MAXIT : CG_BREAKDOWN;
        if (info) {
            for (int j = 0; j < s; ++j) {
                cg_info& o = info[j];
                o.iters = h.k;
                o.status = code;
                o.replacements = h.restarts;
                o.outer = h.rank;
                o.relres_recur = f.nb[j] > 0 ? std::sqrt(h.rr[j]) / f.nb[j] : 0.0;
                o.relres_true = f.nb[j] > 0 ? std::sqrt(f.rr[j]) / f.nb[j] : 0.0;
                o.seconds = ms * 1e-3;
            }
        }
        return code;
    } catch (const HipError& e) {
        return set_error(c, CG_EHIP, std::string("cg_solve_block: ") + e.what + ": " + hipGetErrorString(e.code));
    }
}

}  // extern "C"
