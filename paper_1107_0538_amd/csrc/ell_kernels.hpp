// Standard-form Jacobi-PCG over slices (ell.hpp), for systems that the on-chip
// solver does not hold.  The recurrences, the order of the tests and the state
// block are those of std_kernels.hpp; an iteration is three kernels:
//
//   k_ell_direction  reduce the partials of r'z and r'r, the tests, beta;
//        x += alpha_{k-1} p_{k-1}, p = M^-1 r + beta p
//   k_ell_product    q = A p, partials of p'q
//   k_ell_update     alpha; r -= alpha q; partials of r'z and r'r
//
// x += alpha p of an iteration waits for the next one's direction kernel,
// which reads p anyway (k_ell_flush does it when the iteration stops there),
// and z = M^-1 r is formed where it is used: 12 vectors of N doubles move per
// iteration besides the matrix.  Forming p inside the product's gathers as the
// tile kernels do saves a launch but gathers two vectors: at 128^3 164 us per
// iteration (146 of them the product) against 141 in three kernels (109 + 18 +
// 14), and 196 by tiles; streaming FP32 values 107 against 177.
#pragma once

#include "ell_host.hpp"

namespace jpcg {

// f(s) for the workgroup's slices: a wave takes every kEllWaves-th of the
// workgroup's run; blocks of one XCD own neighbouring runs.
template <typename F>
__device__ __forceinline__ void ell_slices(const EllMap& m, int G, F f)
{
    const int L = logical_of(G), per = (m.S + G - 1) / G;
    const int s1 = min((L + 1) * per, m.S);
    for (int s = L * per + __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave); s < s1; s += kEllWaves) f(s);
}

// The workgroup reduces G interleaved K-tuples in a fixed order; every thread
// gets the sums (contains workgroup barriers).
template <int K>
__device__ __forceinline__ void ell_sums(const double* part, int G, double (&g)[K], double* lds)
{
    grid_sum<kEllBS, K>(part, G, g, lds);
}

// r_out = b - A x (if given): shares of r'r, r'z, b'b.
template <int U>
__device__ __forceinline__ void ell_residual(const EllArgs& a, double* r_out, double& rr, double& rz, double& bb)
{
    const double* __restrict__ x = a.x;
    ell_slices(a.m, a.G, [&](int s) {
        const int lane = threadIdx.x & (kWave - 1), i = s * kEllRows + lane;
        const double ax = ell_row<false, U>(a.m, a.m.val, a.keep, s, lane, x, 0.0);
        if (i < a.m.n) {
            const double bi = a.b[i], ri = bi - ax, zi = a.dinv[i] * ri;
            if (r_out) r_out[i] = ri;
            rr += ri * ri;
            rz += ri * zi;
            bb += bi * bi;
        }
    });
}

template <int U>
__global__ __launch_bounds__(kEllBS) void k_ell_setup(EllArgs a)
{
    __shared__ double lds[kEllWaves * 4];
    double v[3] = {0.0, 0.0, 0.0};
    ell_residual<U>(a, a.r, v[0], v[1], v[2]);
    block_partials<kEllBS, 3>(v, lds, a.part_setup, logical_of(a.G));
}

// One workgroup: the initial tests.
static __global__ __launch_bounds__(kEllBS) void k_ell_begin(EllArgs a, double tol, int maxit)
{
    __shared__ double lds[kEllWaves * 4];
    double g[3];
    ell_sums<3>(a.part_setup, a.G, g, lds);
    const double rr = g[0], nb = sqrt(g[2]), thr = tol * nb;
    if (threadIdx.x != 0) return;
    CgState* st = &a.st->cg;
    st->k = 0;
    st->maxit = maxit;
    st->replacements = 0;
    st->nb = nb;
    st->thr = thr;
    st->rho[1] = g[1];
    st->rr = rr;
    st->rr_true = -1.0;
    st->rr_ref = rr;
    if (a.hist) a.hist[0] = nb > 0.0 ? sqrt(rr) / nb : 0.0;
    st->stop = nb == 0.0 ? STOP_ZERO_RHS : (sqrt(rr) <= thr ? STOP_CONV0 : RUNNING);
    if (nb == 0.0) st->rr_true = 0.0;
    else if (sqrt(rr) <= thr) st->rr_true = rr;
    a.st->pend[0] = a.st->pend[1] = 0;
}

// Iteration k, parity P = k % 2.
static __global__ __launch_bounds__(kEllBS) void k_ell_direction(EllArgs a, int P)
{
    __shared__ double lds[kEllWaves * 4];
    CgState* st = &a.st->cg;
    const int L = logical_of(a.Gu);
    const bool lead = threadIdx.x == 0 && L == 0;
    const int stop = st->stop, km1 = st->k, maxit = st->maxit;
    if (stop != RUNNING) return;
    const double rr_ref = st->rr_ref, thr = st->thr, nb = st->nb, rho_prev = st->rho[P ^ 1], alpha = st->alpha;
    const bool pend = a.st->pend[P ^ 1] != 0;
    double beta = 0.0;
    if (km1 > 0) {
        double g[2];
        ell_sums<2>(a.part_iter, a.Gu, g, lds);
        const double rz = g[0], rr = g[1];
        if (lead) {
            st->rr = rr;
            if (a.hist) a.hist[km1] = sqrt(rr) / nb;
        }
        // The order of the tests: continue-condition (with the reliable
        // updates of the FP32-matrix form), breakdown of r'z, iteration limit.
        int code = RUNNING;
        if (sqrt(rr) <= thr || rr <= a.drop2 * rr_ref) code = STOP_CHECK;
        else if (!(rz > 0.0) || !isfinite(rz)) code = STOP_BREAKDOWN;
        else if (km1 >= maxit) code = STOP_MAXIT;
        if (code != RUNNING) {
            if (lead) st->stop = code;
            return;  // the same decision in every workgroup
        }
        beta = rz / rho_prev;
        if (lead) {
            st->rho[P] = rz;
            st->beta = beta;
        }
    }
    const int rs = min(L * a.R, a.m.n), re = min(rs + a.R, a.m.n);
    for (int i = rs + (int)threadIdx.x; i < re; i += kEllBS) {
        const double zi = a.dinv[i] * a.r[i];
        if (km1 == 0) {
            a.p[i] = zi;
        } else {
            const double pi = a.p[i];
            if (pend) a.x[i] = __builtin_fma(alpha, pi, a.x[i]);
            a.p[i] = __builtin_fma(beta, pi, zi);
        }
    }
}

template <bool M32, int U>
__global__ __launch_bounds__(kEllBS) void k_ell_product(EllArgs a)
{
    __shared__ double lds[kEllWaves * 4];
    if (a.st->cg.stop != RUNNING) return;
    const double* __restrict__ p = a.p;
    double v[1] = {0.0};
    ell_slices(a.m, a.G, [&](int s) {
        const int lane = threadIdx.x & (kWave - 1), i = s * kEllRows + lane;
        const double pi = p[min(i, a.m.n - 1)];
        double y;
        if constexpr (M32) y = ell_row<true, U>(a.m, a.m.val32, a.keep, s, lane, p, pi);
        else y = ell_row<false, U>(a.m, a.m.val, a.keep, s, lane, p, 0.0);
        if (i < a.m.n) {
            if constexpr (M32) y = __builtin_fma(a.rowsum[i], pi, y);
            a.q[i] = y;
            v[0] += pi * y;
        }
    });
    block_partials<kEllBS, 1>(v, lds, a.part_sig, logical_of(a.G));
}

static __global__ __launch_bounds__(kEllBS) void k_ell_update(EllArgs a, int P)
{
    __shared__ double lds[kEllWaves * 4];
    CgState* st = &a.st->cg;
    const int stop = st->stop;
    const double rho = st->rho[P];
    const int L = logical_of(a.Gu);
    const int rs = min(L * a.R, a.m.n), re = min(rs + a.R, a.m.n);
    if (stop != RUNNING) return;
    double g[1];
    ell_sums<1>(a.part_sig, a.G, g, lds);
    const double sigma = g[0];
    __syncthreads();
    const bool lead = threadIdx.x == 0 && L == 0;
    if (!(sigma > 0.0) || !isfinite(sigma)) {
        if (lead) {
            st->stop = STOP_BREAKDOWN;
            a.st->pend[P ^ 1] = 0;  // the direction kernel has done it
        }
        return;
    }
    const double alpha = rho / sigma;
    double v[2] = {0.0, 0.0};
    for (int i = rs + (int)threadIdx.x; i < re; i += kEllBS) {
        const double ri = __builtin_fma(-alpha, a.q[i], a.r[i]);
        const double zi = a.dinv[i] * ri;
        a.r[i] = ri;
        v[0] += ri * zi;
        v[1] += ri * ri;
    }
    block_partials<kEllBS, 2>(v, lds, a.part_iter, L);
    if (lead) {
        st->k = st->k + 1;
        st->sigma = sigma;
        st->alpha = alpha;
        a.st->pend[P] = 1;
    }
}

// x += alpha_k p_k where the iteration stopped before its next direction.
static __global__ __launch_bounds__(kEllBS) void k_ell_flush(EllArgs a, int P)
{
    if (!a.st->pend[P]) return;
    const double alpha = a.st->cg.alpha;
    const double* __restrict__ p = a.p;
    for (int i = blockIdx.x * kEllBS + threadIdx.x; i < a.m.n; i += gridDim.x * kEllBS)
        a.x[i] = __builtin_fma(alpha, p[i], a.x[i]);
}
static __global__ void k_ell_flushed(EllArgs a) { a.st->pend[0] = a.st->pend[1] = 0; }

// r = b - A x with `replace`; partials of r'z and r'r.
template <int U>
__global__ __launch_bounds__(kEllBS) void k_ell_check(EllArgs a, int replace)
{
    __shared__ double lds[kEllWaves * 4];
    double rr = 0.0, rz = 0.0, bb = 0.0;
    ell_residual<U>(a, replace ? a.r : nullptr, rr, rz, bb);
    double v[2] = {rz, rr};
    block_partials<kEllBS, 2>(v, lds, a.part_chk, logical_of(a.G));
}

// One workgroup: accept the solve, or resume with the replaced residual, whose
// sums the next direction kernel finds where B leaves its partials; with
// report only ||b - A x||^2 is recorded.
static __global__ __launch_bounds__(kEllBS) void k_ell_decide(EllArgs a, int report)
{
    __shared__ double lds[kEllWaves * 4];
    double g[2];
    ell_sums<2>(a.part_chk, a.G, g, lds);
    CgState* st = &a.st->cg;
    const bool pass = sqrt(g[1]) <= st->thr;
    for (int j = threadIdx.x; j < a.Gu; j += kEllBS) {
        a.part_iter[2 * j] = j == 0 ? g[0] : 0.0;
        a.part_iter[2 * j + 1] = j == 0 ? g[1] : 0.0;
    }
    if (threadIdx.x == 0) {
        if (report) {
            st->rr_true = g[1];
        } else if (pass) {
            st->stop = STOP_CONVERGED;
            st->rr_true = g[1];
        } else {
            st->stop = RUNNING;
            st->replacements += 1;
            st->rr_ref = g[1];
        }
    }
}

// y = A x; a workgroup is one wave and one slice, as nothing is shared and a
// free wave slot is filled at once: at 51^3 7.5 us in blocks of 64, 7.8 of 128,
// 8.4 of 256, 10.0 of 512; from 64^3 on no difference.
template <int U>
__global__ __launch_bounds__(kEllRows) void k_ell_spmv(EllMap m, int keep, int G, const double* __restrict__ x,
                                                       double* __restrict__ y)
{
    const int s = logical_of(G);
    if (s >= m.S) return;
    const int lane = threadIdx.x, i = s * kEllRows + lane;
    const double t = ell_row<false, U>(m, m.val, keep, s, lane, x, 0.0);
    if (i < m.n) y[i] = t;
}

}  // namespace jpcg
