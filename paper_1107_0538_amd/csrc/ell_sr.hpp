// Single-reduction Jacobi-PCG (sr_kernels.hpp: the recurrences, the order of
// the tests, the state block and the restart after a replacement) over slices,
// in two kernels an iteration:
//
//   k_ell_sr_update   reduce the partials, the tests, alpha and beta; p, s, x, r
//                     and u = M^-1 r of the own rows; partials of r'u, r'r,
//                     p's and u's
//   k_ell_sr_product  w = A u; partials of w'u and p'w
//
// Forming u inside the gathers, as the one kernel over tiles does, fetches 32
// bytes per entry; u stored once moves 14 vectors of N doubles an iteration
// besides the matrix.  A solve at 66^3, 84^3, 96^3 and 118^3 takes 13.9, 27.9,
// 46.1 and 110 ms, over tiles 17.6, 36.7, 70.0 and 155.
#pragma once

#include "ell_kernels.hpp"
#include "sr_kernels.hpp"

namespace jpcg {

// Partials of the update kernel: r'u, r'r, p's, u's.
constexpr int kEllSrPart = 4;

// K_k, parity P = k % 2; the update kernel's partials are in part[parity].
static __global__ __launch_bounds__(kEllBS) void k_ell_sr_update(EllSrArgs a, int P)
{
    __shared__ double lds[kEllWaves * 4];
    SrState* st = a.st;
    const int Q = P ^ 1, L = logical_of(a.Gu);
    const bool lead = threadIdx.x == 0 && L == 0;
    const int stop = st->stop, maxit = st->maxit, km1 = st->kk[Q];
    if (stop != RUNNING) return;
    const double thr = st->thr, nb = st->nb, gam2 = st->gam[Q];
    double g[kEllSrPart], h[2];
    ell_sums<kEllSrPart>(a.part[Q], a.Gu, g, lds);
    __syncthreads();
    ell_sums<2>(a.part_w, a.G, h, lds);
    __syncthreads();
    const double gam = g[0], rr = g[1], delta = h[0];
    if (lead) {
        st->rr = rr;
        if (a.hist) a.hist[km1] = sqrt(rr) / nb;
    }
    // The oracle's order: continue-condition, breakdown of gamma, iteration
    // limit, then breakdown of sigma at the top of the next iteration.
    int code = RUNNING;
    double beta = 0.0, sigma = delta;
    if (sqrt(rr) <= thr) code = STOP_CHECK;
    else if (!(gam > 0.0) || !isfinite(gam)) code = STOP_BREAKDOWN;
    else if (km1 >= maxit) code = STOP_MAXIT;
    else {
        if (km1 > 0) {
            beta = gam / gam2;
            sigma = delta + beta * (g[3] + h[1]) + beta * beta * g[2];
        }
        if (!(sigma > 0.0) || !isfinite(sigma)) code = STOP_BREAKDOWN;
    }
    if (code != RUNNING) {
        if (lead) {
            st->k_done = km1;
            st->stop = code;
        }
        return;  // the same decision in every workgroup
    }
    const double alpha = gam / sigma;
    double v[kEllSrPart] = {0.0, 0.0, 0.0, 0.0};
    const int rs = min(L * a.R, a.m.n), re = min(rs + a.R, a.m.n);
    for (int i = rs + (int)threadIdx.x; i < re; i += kEllBS) {
        const double d = a.dinv[i], r0 = a.r[i];
        const double pi = __builtin_fma(beta, a.p[i], d * r0);
        const double si = __builtin_fma(beta, a.s[i], a.w[i]);
        const double ri = __builtin_fma(-alpha, si, r0);
        const double ui = d * ri;
        a.x[i] = __builtin_fma(alpha, pi, a.x[i]);
        a.p[i] = pi;
        a.s[i] = si;
        a.r[i] = ri;
        a.u[i] = ui;
        v[0] += ri * ui;
        v[1] += ri * ri;
        v[2] += pi * si;
        v[3] += ui * si;
    }
    block_partials<kEllBS, kEllSrPart>(v, lds, a.part[P], L);
    if (lead) {
        st->kk[P] = km1 + 1;
        st->gam[P] = gam;
    }
}

// w = A u; partials of w'u and p'w.
template <int U>
__global__ __launch_bounds__(kEllBS) void k_ell_sr_product(EllSrArgs a)
{
    __shared__ double lds[kEllWaves * 4];
    if (a.st->stop != RUNNING) return;
    const double* __restrict__ u = a.u;
    double v[2] = {0.0, 0.0};
    ell_slices(a.m, a.G, [&](int s) {
        const int lane = threadIdx.x & (kWave - 1), i = s * kEllRows + lane, j = min(i, a.m.n - 1);
        const double ui = u[j], pi = a.p[j];
        const double y = ell_row<false, U>(a.m, a.m.val, a.keep, s, lane, u, 0.0);
        if (i < a.m.n) {
            a.w[i] = y;
            v[0] += y * ui;
            v[1] += pi * y;
        }
    });
    block_partials<kEllBS, 2>(v, lds, a.part_w, logical_of(a.G));
}

// ||b - A x||^2 (part_chk: with b'b); with replace the residual replaces r,
// with setup p and s are cleared too.
template <int U>
__global__ __launch_bounds__(kEllBS) void k_ell_sr_residual(EllSrArgs a, int replace, int setup)
{
    __shared__ double lds[kEllWaves * 4];
    const double* __restrict__ x = a.x;
    double v[2] = {0.0, 0.0};
    ell_slices(a.m, a.G, [&](int s) {
        const int lane = threadIdx.x & (kWave - 1), i = s * kEllRows + lane;
        const double ax = ell_row<false, U>(a.m, a.m.val, a.keep, s, lane, x, 0.0);
        if (i < a.m.n) {
            const double bi = a.b[i], ri = bi - ax;
            if (replace) a.r[i] = ri;
            if (setup) a.p[i] = a.s[i] = 0.0;
            v[0] += ri * ri;
            v[1] += bi * bi;
        }
    });
    block_partials<kEllBS, 2>(v, lds, a.part_chk, logical_of(a.G));
}

// One workgroup: the initial tests.
static __global__ __launch_bounds__(kEllBS) void k_ell_sr_begin(EllSrArgs a, double tol, int maxit)
{
    __shared__ double lds[kEllWaves * 4];
    double g[2];
    ell_sums<2>(a.part_chk, a.G, g, lds);
    if (threadIdx.x != 0) return;
    const double rr = g[0], nb = sqrt(g[1]), thr = tol * nb;
    SrState* st = a.st;
    st->kk[0] = st->kk[1] = 0;
    st->k_done = 0;
    st->maxit = maxit;
    st->replacements = 0;
    st->nb = nb;
    st->thr = thr;
    st->rr = rr;
    st->rr_true = -1.0;
    if (a.hist) a.hist[0] = nb > 0.0 ? sqrt(rr) / nb : 0.0;
    st->stop = nb == 0.0 ? STOP_ZERO_RHS : (sqrt(rr) <= thr ? STOP_CONV0 : RUNNING);
    if (nb == 0.0) st->rr_true = 0.0;
    else if (sqrt(rr) <= thr) st->rr_true = rr;
}

// u = M^-1 r with its partials in part[P]; s = A p first if `restart` (after a
// replacement; at the start p and s are zero).
template <int U>
__global__ __launch_bounds__(kEllBS) void k_ell_sr_start(EllSrArgs a, int P, int restart)
{
    __shared__ double lds[kEllWaves * 4];
    if (a.st->stop != RUNNING) return;
    const double* __restrict__ p = a.p;
    double v[kEllSrPart] = {0.0, 0.0, 0.0, 0.0};
    ell_slices(a.m, a.Gu, [&](int s) {
        const int lane = threadIdx.x & (kWave - 1), i = s * kEllRows + lane;
        double si = 0.0;
        if (restart) si = ell_row<false, U>(a.m, a.m.val, a.keep, s, lane, p, 0.0);
        if (i < a.m.n) {
            const double ri = a.r[i], ui = a.dinv[i] * ri;
            a.u[i] = ui;
            if (restart) a.s[i] = si;
            v[0] += ri * ui;
            v[1] += ri * ri;
            v[2] += p[i] * si;
            v[3] += ui * si;
        }
    });
    block_partials<kEllBS, kEllSrPart>(v, lds, a.part[P], logical_of(a.Gu));
}

// One workgroup: accept, or resume after a replacement; with report only
// ||b - A x||^2 is recorded.
static __global__ __launch_bounds__(kEllBS) void k_ell_sr_decide(EllSrArgs a, int report)
{
    __shared__ double lds[kEllWaves * 4];
    double g[2];
    ell_sums<2>(a.part_chk, a.G, g, lds);
    if (threadIdx.x != 0) return;
    SrState* st = a.st;
    if (report) {
        st->rr_true = g[0];
    } else if (sqrt(g[0]) <= st->thr) {
        st->stop = STOP_CONVERGED;
        st->rr_true = g[0];
    } else {
        st->stop = RUNNING;
        st->replacements += 1;
    }
}

}  // namespace jpcg
