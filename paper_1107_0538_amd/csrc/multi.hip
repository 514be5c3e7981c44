// Multi-RHS Jacobi-PCG: s <= 64 independent CG recurrences (one per column of
// a row-major N x s block) sharing one sparse product per iteration.
//
// Each column follows the FP64 oracle's loop exactly; the columns only share
// launches.  spmm's column j equals the sequential CSR product (spmm.hpp).
//
// Per iteration, all captured in hipGraph chunks:
//   k_mr_direction  x_j += alpha_j p_j of the iteration before, then
//                   p_j = z_j + beta_j p_j (active) or z_j (first step), with
//                   z = M^-1 r formed here; frozen columns keep their p
//   k_mr_product    q = A p, partials of p_j'q_j
//   k_mr_scalars    one workgroup per column: sigma_j, alpha_j, breakdown
//   k_mr_update     r -= alpha q, partials of r'z, r'r
//   k_mr_scalars    one workgroup per column: continue-condition, breakdown,
//                   limit, beta
// An iteration moves ten blocks of N x s besides the matrix (x waits for the
// pass that reads p anyway, z is not stored); 51^3 with 64 columns takes 169 us
// an iteration (direction 51, product 74, update 31, scalars 5 each) where
// twelve and a product of 204 us took 354.
// A column whose recurrence residual passes is frozen and waits; when no
// column is active the host brings x up to date (k_mr_flush), runs one
// true-residual check for all waiting columns, exactly the oracle's check,
// and resumes replaced ones.  Each column's per-workgroup partials are
// reduced by that column's own workgroup of the scalar kernel, in a fixed
// order; whether any column is still active is read from the 64 statuses by
// every kernel that needs it.
#include <algorithm>
#include <cstddef>
#include <cmath>
#include <cstring>
#include <vector>

#include "spmm.hpp"

namespace jpcg {

enum ColStatus : int {
    COL_ACTIVE = 0,
    COL_PENDING = 1,  // recurrence residual passed; true residual not yet checked
    COL_CONVERGED = 2,
    COL_MAXIT = 3,
    COL_BREAKDOWN = 4,
    COL_ZERO = 5,     // b_j = 0
    COL_UNUSED = 6,   // lane >= s
};

constexpr int kCols = 64;

struct MrState {
    int kk;            // iterations completed
    int ran;           // the last direction kernel found an active column
    int pad[2];
    int status[kCols];
    int iters[kCols];
    int repl[kCols];
    int first[kCols];  // next direction step is the first for this column (p = z)
    int pend[kCols];   // x += alpha p is still to be done
    double rho[kCols];
    double alpha[kCols];
    double beta[kCols];
    double nb[kCols];
    double thr[kCols];
    double rr[kCols];
    double rr_true[kCols];
};

template <typename T>
struct MrArgs {
    RunMap<T> m;
    int n, s;
    const T* __restrict__ dinv;
    const T* B;
    T* X;
    T* R;
    T* P;
    T* Q;
    int G;         // workgroups of the product kernels
    int Gv;        // of the elementwise kernels
    int rows;      // rows per workgroup of the elementwise kernels
    double* part;  // [3][64][G or Gv]
    MrState* st;
    int maxit;
    double tol;
    int confirm;   // 1: a passed recurrence test is confirmed on b - A x; 0: it ends the column
};

constexpr int kMrBS = 256;
static_assert(kMrBS == kSpmmBS, "the product kernels share the blocks' reduction");

// The block's sums of K quantities per column, given per wave in lds, to
// part[k][column][L of G].
template <int K>
__device__ __forceinline__ void mr_write_partials(const double (&lds)[kMrBS / kWave][K][kWave], int s, double* part,
                                                  int L, int G)
{
    __syncthreads();
    for (int e = threadIdx.x; e < K * kWave; e += kMrBS) {
        const int k = e / kWave, j = e % kWave;
        if (j >= s) continue;
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kMrBS / kWave; ++w) t += lds[w][k][j];
        part[(size_t)(k * kWave + j) * G + L] = t;
    }
}

// From the product's lanes (v[k][0]: the lane's first column, v[k][1]: its second).
template <int K>
__device__ __forceinline__ void mr_product_partials(double (&v)[K][2], const SpmmLane& l, double* part, int G)
{
    __shared__ double lds[kMrBS / kWave][K][kWave];
    const int w = threadIdx.x / kWave;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const double a = v[k][0] + __shfl_xor(v[k][0], 32), b = v[k][1] + __shfl_xor(v[k][1], 32);
        if (l.half == 0) {
            if (l.own1) lds[w][k][l.c] = a;
            if (l.own2) lds[w][k][l.c + 1] = b;
        }
    }
    mr_write_partials<K>(lds, l.s, part, (int)blockIdx.x, G);
}

// The elementwise kernels' lanes: V neighbouring columns of a row (2 where s is
// even, 16-byte accesses; else 1), the least power of two of lanes that holds
// a row.
template <int V>
struct MrLane {
    int s, P, c, row;  // columns, lanes per row, first column, row of the workgroup's step
    bool used;
    __device__ explicit MrLane(int s_) : s(s_), P(1)
    {
        while (P * V < s) P *= 2;
        const int t = threadIdx.x & (P - 1);
        c = t * V;
        used = c < s;
        row = threadIdx.x / P;
    }
    __device__ int step() const { return kMrBS / P; }
    template <bool STREAM = false, typename T>
    __device__ void load(const T* p, size_t i, T (&x)[V]) const
    {
        typedef T vec __attribute__((ext_vector_type(V)));
        vec v;
        if constexpr (STREAM) v = __builtin_nontemporal_load((const vec*)(p + i * s + c));
        else v = *(const vec*)(p + i * s + c);
#pragma unroll
        for (int u = 0; u < V; ++u) x[u] = v[u];
    }
    template <bool STREAM = false, typename T>
    __device__ void store(T* p, size_t i, const T (&x)[V]) const
    {
        typedef T vec __attribute__((ext_vector_type(V)));
        vec v;
#pragma unroll
        for (int u = 0; u < V; ++u) v[u] = x[u];
        if constexpr (STREAM) __builtin_nontemporal_store(v, (vec*)(p + i * s + c));
        else *(vec*)(p + i * s + c) = v;
    }
    template <int K>
    __device__ void partials(double (&v)[K][V], double* part, int L, int G) const
    {
        __shared__ double lds[kMrBS / kWave][K][kWave];
        const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int u = 0; u < V; ++u) {
                double t = v[k][u];
                for (int off = P; off < kWave; off *= 2) t += __shfl_xor(t, off);
                if (lane < P && used) lds[w][k][c + u] = t;
            }
        mr_write_partials<K>(lds, s, part, L, G);
    }
};

// True in every thread if some column is active (each wave reads the 64
// statuses once).
__device__ __forceinline__ bool mr_any_active(const MrState* st)
{
    const int lane = threadIdx.x & (kWave - 1);
    return __ballot(st->status[lane] == COL_ACTIVE) != 0ull;
}

// Residual R = B - A X and partials (r'r, r'z, b'b) per column.  mode 0: setup
// (every column), 1: check (only pending columns are rewritten), 2: report
// (nothing is written but the partials).
template <SpmmKind KIND, typename T>
__global__ __launch_bounds__(kMrBS) void k_mr_residual(MrArgs<T> a, int mode)
{
    const SpmmLane l(a.s);
    auto write = [&](int j) { return mode == 0 || (mode == 1 && a.st->status[j] == COL_PENDING); };
    const bool w1 = l.own1 && write(l.c), w2 = l.own2 && write(l.c + 1);
    double v[3][2] = {};
    auto take = [&](size_t i, int u, bool wr, T bi, T ax) {
        const T ri = bi - ax, zi = a.dinv[i] * ri;
        if (wr) a.R[i * a.s + l.c + u] = ri;
        v[0][u] += (double)ri * (double)ri;
        v[1][u] += (double)ri * (double)zi;
        v[2][u] += (double)bi * (double)bi;
    };
    spmm_rows<false, KIND, T>(
        a.m, a.X, l, a.G, [&](int i) { return l.load(a.B, i); },
        [&](int i, T y1, T y2, Pair<T> b) {
            take(i + l.half, 0, w1, b.x, y1);
            take(i + l.half, 1, w2, b.y, y2);
        },
        [&](int i, T y) {
            const T b = a.B[(size_t)i * a.s + l.column()];
            if (l.half == 0) take(i, 0, w1, b, y);
            else if (a.s > 1) take(i, 1, w2, b, y);
        });
    mr_product_partials<3>(v, l, a.part, a.G);
}

// x += alpha p where the last iteration left it; p = z + beta p (active), z
// (first step), unchanged (frozen).  Bound by memory: five blocks, 340 MB at
// 51^3 with 64 columns in 51 us.
template <int V, bool S, typename T>
__global__ __launch_bounds__(kMrBS) void k_mr_direction(MrArgs<T> a)
{
    MrState* st = a.st;
    const bool any = mr_any_active(st);
    const int L = xcd_logical_block((int)blockIdx.x, a.Gv);
    if (L == 0 && threadIdx.x == 0) st->ran = any;
    if (!any) return;
    const MrLane<V> l(a.s);
    if (!l.used) return;
    bool active[V], first[V], pend[V], work = false, late = false;
    T alpha[V], beta[V];
#pragma unroll
    for (int u = 0; u < V; ++u) {
        const int j = l.c + u;
        active[u] = st->status[j] == COL_ACTIVE;
        first[u] = st->first[j] != 0;
        pend[u] = st->pend[j] != 0;
        alpha[u] = (T)st->alpha[j];
        beta[u] = (T)st->beta[j];
        work = work || active[u] || pend[u];
        late = late || pend[u];
    }
    if (!work) return;
    const int rs = min(L * a.rows, a.n), re = min(rs + a.rows, a.n);
    for (int i = rs + l.row; i < re; i += l.step()) {
        T r[V], p[V];
        l.template load<S>(a.R, i, r);
        l.load(a.P, i, p);
        const T d = a.dinv[i];
        if (late) {
            T x[V];
            l.template load<S>(a.X, i, x);
#pragma unroll
            for (int u = 0; u < V; ++u) x[u] = pend[u] ? fma_t(alpha[u], p[u], x[u]) : x[u];
            l.template store<S>(a.X, i, x);
        }
#pragma unroll
        for (int u = 0; u < V; ++u) {
            const T z = d * r[u];
            p[u] = active[u] ? (first[u] ? z : fma_t(beta[u], p[u], z)) : p[u];
        }
        l.store(a.P, i, p);
    }
}

// x += alpha p where the iterations stopped before their next direction.
template <typename T>
__global__ __launch_bounds__(kMrBS) void k_mr_flush(MrArgs<T> a)
{
    const MrLane<1> l(a.s);
    if (!l.used || !a.st->pend[l.c]) return;
    const T alpha = (T)a.st->alpha[l.c];
    const int L = xcd_logical_block((int)blockIdx.x, a.Gv), rs = min(L * a.rows, a.n), re = min(rs + a.rows, a.n);
    for (int i = rs + l.row; i < re; i += l.step()) {
        T x[1], p[1];
        l.load(a.X, i, x);
        l.load(a.P, i, p);
        x[0] = fma_t(alpha, p[0], x[0]);
        l.store(a.X, i, x);
    }
}
static __global__ void k_mr_flushed(MrState* st) { st->pend[threadIdx.x] = 0; }

// q = A p; partials of p'q.
template <SpmmKind KIND, typename T>
__global__ __launch_bounds__(kMrBS, KIND == SPMM_SINGLE ? spmm_waves(KIND) : 5) void k_mr_product(MrArgs<T> a)
{
    if (!mr_any_active(a.st)) return;
    const SpmmLane l(a.s);
    double v[1][2] = {};
    spmm_rows<sizeof(T) == 4, KIND, T>(
        a.m, a.P, l, a.G, [&](int i) { return l.load(a.P, i); },
        [&](int i, T q1, T q2, Pair<T> p) {
            l.store(a.Q, i, q1, q2);
            v[0][0] += (double)p.x * (double)q1;
            v[0][1] += (double)p.y * (double)q2;
        },
        [&](int i, T q) {
            const size_t o = (size_t)i * a.s + l.column();
            const double pq = (double)a.P[o] * (double)q;
            if (l.own()) a.Q[o] = q;
            if (l.half == 0) v[0][0] += pq;
            else v[0][1] += pq;
        });
    mr_product_partials<1>(v, l, a.part, a.G);
}

// r -= alpha q for active columns; partials of r'z, r'r.  Three blocks, 204 MB in
// 31 us.
template <int V, bool S, typename T>
__global__ __launch_bounds__(kMrBS) void k_mr_update(MrArgs<T> a)
{
    MrState* st = a.st;
    if (!mr_any_active(st)) return;
    const int L = xcd_logical_block((int)blockIdx.x, a.Gv);
    if (L == 0 && threadIdx.x == 0) st->kk += 1;  // this iteration is being done
    const MrLane<V> l(a.s);
    bool active[V], work = false;
    T alpha[V];
#pragma unroll
    for (int u = 0; u < V; ++u) {
        const int j = l.used ? l.c + u : 0;
        active[u] = l.used && st->status[j] == COL_ACTIVE;
        alpha[u] = (T)st->alpha[j];
        work = work || active[u];
    }
    double v[2][V] = {};
    if (work) {
        const int rs = min(L * a.rows, a.n), re = min(rs + a.rows, a.n);
        for (int i = rs + l.row; i < re; i += l.step()) {
            T r[V], q[V];
            l.template load<S>(a.R, i, r);
            l.load(a.Q, i, q);
            const T d = a.dinv[i];
#pragma unroll
            for (int u = 0; u < V; ++u) {
                r[u] = active[u] ? fma_t(-alpha[u], q[u], r[u]) : r[u];
                const T z = d * r[u];
                v[0][u] += (double)r[u] * (double)z;
                v[1][u] += (double)r[u] * (double)r[u];
            }
            l.template store<S>(a.R, i, r);
        }
    }
    l.partials(v, a.part, L, a.Gv);
}

enum MrPhase : int { MR_SETUP = 0, MR_SIGMA = 1, MR_ITER = 2, MR_CHECK = 3, MR_REPORT = 4 };

// Column j's sums of the G per-workgroup partials of K quantities, in a fixed
// order; the totals are returned in every thread.
template <int BS, int K>
__device__ __forceinline__ void mr_column_sum(const double* part, int G, int j, double (&out)[K], double* lds)
{
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = 0.0;
    for (int g = threadIdx.x; g < G; g += BS) {
#pragma unroll
        for (int k = 0; k < K; ++k) out[k] += part[(size_t)(k * kWave + j) * G + g];
    }
    block_sum<BS, K>(out, lds);
}

// The per-column scalar steps: workgroup j owns column j's state.
template <typename T>
__global__ __launch_bounds__(256) void k_mr_scalars(MrArgs<T> a, int phase)
{
    __shared__ double lds[(256 / kWave) * 3];
    MrState* st = a.st;
    const int j = blockIdx.x;
    if (phase == MR_SETUP && j == 0 && threadIdx.x == 0) st->kk = 0;
    if (j >= a.s) {
        if (phase == MR_SETUP && threadIdx.x == 0) st->status[j] = COL_UNUSED;
        return;
    }
    int status = st->status[j];
    if (phase == MR_SIGMA && status != COL_ACTIVE && st->ran && threadIdx.x == 0) st->pend[j] = 0;
    if ((phase == MR_SIGMA || phase == MR_ITER) && status != COL_ACTIVE) return;
    if (phase == MR_CHECK && status != COL_PENDING) return;
    double g[3] = {0.0, 0.0, 0.0};
    if (phase == MR_SIGMA) {
        double t[1];
        mr_column_sum<256, 1>(a.part, a.G, j, t, lds);
        g[0] = t[0];
    } else if (phase == MR_ITER) {
        double t[2];
        mr_column_sum<256, 2>(a.part, a.Gv, j, t, lds);
        g[0] = t[0];
        g[1] = t[1];
    } else {
        mr_column_sum<256, 3>(a.part, a.G, j, g, lds);
    }
    if (threadIdx.x != 0) return;
    if (phase == MR_SETUP) {
        // g = (r'r, r'z, b'b) of r0
        st->repl[j] = 0;
        st->iters[j] = 0;
        st->first[j] = 1;
        st->beta[j] = 0.0;
        st->alpha[j] = 0.0;
        st->pend[j] = 0;
        const double nb = sqrt(g[2]);
        st->nb[j] = nb;
        st->thr[j] = a.tol * nb;
        st->rr[j] = g[0];
        st->rho[j] = g[1];
        st->rr_true[j] = -1.0;
        if (nb == 0.0) {
            status = COL_ZERO;
            st->rr_true[j] = 0.0;
        } else if (sqrt(g[0]) <= a.tol * nb) {
            status = COL_CONVERGED;
            st->rr_true[j] = g[0];
        } else {
            status = COL_ACTIVE;
        }
    } else if (phase == MR_SIGMA) {
        const double sigma = g[0];
        const bool ok = sigma > 0.0 && isfinite(sigma);
        if (ok) st->alpha[j] = st->rho[j] / sigma;
        else status = COL_BREAKDOWN;
        st->pend[j] = ok;  // the direction kernel has done the last one
    } else if (phase == MR_ITER) {
        // g = (r'z, r'r) after the update: the oracle's order of tests.
        st->iters[j] += 1;
        st->first[j] = 0;
        st->rr[j] = g[1];
        if (sqrt(g[1]) <= st->thr[j]) {
            status = a.confirm ? COL_PENDING : COL_CONVERGED;
            if (!a.confirm) st->rr_true[j] = g[1];
        } else if (!(g[0] > 0.0) || !isfinite(g[0])) {
            status = COL_BREAKDOWN;
        } else if (st->iters[j] >= a.maxit) {
            status = COL_MAXIT;
        } else {
            st->beta[j] = g[0] / st->rho[j];
            st->rho[j] = g[0];
        }
    } else if (phase == MR_CHECK) {
        // g = (r'r, r'z, b'b) of the true residual; r, z were replaced for pending columns.
        if (sqrt(g[0]) <= st->thr[j]) {
            status = COL_CONVERGED;
            st->rr_true[j] = g[0];
        } else if (!(g[1] > 0.0) || !isfinite(g[1])) {
            status = COL_BREAKDOWN;
        } else if (st->iters[j] >= a.maxit) {
            status = COL_MAXIT;
        } else {
            status = COL_ACTIVE;
            st->repl[j] += 1;
            st->beta[j] = g[1] / st->rho[j];
            st->rho[j] = g[1];
        }
    } else {  // MR_REPORT: true residual of the returned x for every column
        if (status != COL_ZERO) st->rr_true[j] = g[0];
    }
    st->status[j] = status;
}

// Mixed form, outer step: B32 = R64 / ||r_j|| for the columns still active
// in the FP64 state (0 for the others), X32 = 0.
__global__ void k_mr_scale(int n, int s, const double* __restrict__ r64, const MrState* st64,
                           float* __restrict__ b32, float* __restrict__ x32)
{
    const int lane = threadIdx.x & (kWave - 1);
    if (lane >= s) return;
    const bool active = st64->status[lane] == COL_ACTIVE;
    const double nr = sqrt(st64->rr[lane]);
    const double inv = active && nr > 0.0 ? 1.0 / nr : 0.0;
    for (int i = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; i < n; i += gridDim.x * (blockDim.x / kWave)) {
        const size_t o = (size_t)i * s + lane;
        b32[o] = (float)(r64[o] * inv);
        x32[o] = 0.0f;
    }
}

// Mixed form: X64 += ||r_j|| X32 for the columns that were active.
__global__ void k_mr_fold(int n, int s, double* __restrict__ x64, const float* __restrict__ x32, const MrState* st64)
{
    const int lane = threadIdx.x & (kWave - 1);
    if (lane >= s || st64->status[lane] != COL_ACTIVE) return;
    const double nr = sqrt(st64->rr[lane]);
    for (int i = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; i < n; i += gridDim.x * (blockDim.x / kWave)) {
        const size_t o = (size_t)i * s + lane;
        x64[o] = fma(nr, (double)x32[o], x64[o]);
    }
}

// x_j = 0 for columns with b_j = 0.
template <typename T>
__global__ void k_mr_zero_cols(MrArgs<T> a)
{
    const int lane = threadIdx.x & (kWave - 1);
    if (lane >= a.s || a.st->status[lane] != COL_ZERO) return;
    for (int i = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; i < a.n;
         i += gridDim.x * (blockDim.x / kWave))
        a.X[(size_t)i * a.s + lane] = T(0);
}

}  // namespace jpcg

// Multi-RHS solver state hanging off a context, for one block width s and
// one precision (FP64, or the FP32 inner solver of the mixed form).
struct cg_multi {
    int s = 0, chunk = 0;
    bool stream = false;   // R and X pass the last-level cache by
    bool fp32 = false;
    void* work = nullptr;  // R, P, Q, and the solver's own B, X: 5 N s values
    double* part = nullptr;
    jpcg::MrState* st = nullptr;
    jpcg::MrState* hst = nullptr;
    const void *product = nullptr, *residual = nullptr;
    hipGraphExec_t exec = nullptr;
    hipEvent_t ev = nullptr;
    jpcg::MrArgs<double> args{};
    jpcg::MrArgs<float> args32{};
};

namespace jpcg {

static void destroy_multi(cg_multi* m)
{
    if (!m) return;
    if (m->exec) (void)hipGraphExecDestroy(m->exec);
    if (m->ev) (void)hipEventDestroy(m->ev);
    if (m->work) (void)hipFree(m->work);
    if (m->part) (void)hipFree(m->part);
    if (m->st) (void)hipFree(m->st);
    if (m->hst) (void)hipHostFree(m->hst);
    delete m;
}

static void mr_launch(const void* fn, int grid, int bs, hipStream_t st, void** args)
{
    JPCG_HIP(hipLaunchKernel(fn, dim3(grid), dim3(bs), args, 0, st));
}

template <typename T>
static MrArgs<T>& margs(cg_multi* m);
template <>
MrArgs<double>& margs<double>(cg_multi* m) { return m->args; }
template <>
MrArgs<float>& margs<float>(cg_multi* m) { return m->args32; }

// The words of spmm.hpp's fours of rows; found: how many are to be streams, how
// many of those hold a row longer than half a wave, and how many are runs.
static __global__ __launch_bounds__(256) void k_find_runs(int n, const int* __restrict__ rowptr,
                                                          const int* __restrict__ col, int* __restrict__ runs, int* found)
{
    const int g = blockIdx.x * 256 + threadIdx.x, i0 = g * kRunRows;
    if (i0 >= n) return;
    const int rows = min(kRunRows, n - i0), k0 = rowptr[i0], len = rowptr[i0 + 1] - k0;
    int most = len;
    for (int r = 1; r < rows; ++r) most = max(most, rowptr[i0 + r + 1] - rowptr[i0 + r]);
    bool ok = rows == kRunRows && len % 3 == 0 && len <= kSpmmShort;
    for (int r = 1; ok && r < kRunRows; ++r) ok = rowptr[i0 + r + 1] - rowptr[i0 + r] == len;
    for (int e = 0; ok && e < len; ++e) {
        const int c = col[k0 + e / 3 * 3] + e % 3;
        for (int r = 0; ok && r < kRunRows; ++r) ok = col[k0 + r * len + e] == c + r;
    }
    const int own = rowptr[i0 + rows] - k0;
    const bool stream = most > kSpmmShort || rows * most > kSpmmPadding * own + 8;
    runs[g] = ok && len ? len : stream ? SPMM_STREAM : SPMM_EVEN;
    const int uneven = __popcll(__ballot(runs[g] < 0)), longer = __popcll(__ballot(most > kSpmmShort));
    const int whole = __popcll(__ballot(runs[g] > 0));
    if ((threadIdx.x & (kWave - 1)) == 0) {
        if (uneven) atomicAdd(&found[0], uneven);
        if (longer) atomicAdd(&found[1], longer);
        if (whole) atomicAdd(&found[2], whole);
    }
}

void make_runs(cg_ctx* c, int* found)
{
    const int fours = (c->n + kRunRows - 1) / kRunRows;
    JPCG_HIP(hipMalloc(&c->runs, sizeof(int) * fours));
    k_find_runs<<<(fours + 255) / 256, 256, 0, c->stream>>>(c->n, c->rowptr, c->col, c->runs, found);
    JPCG_HIP(hipGetLastError());
}

// A few fours of unequal rows, as at the ends of a lattice's lines, may well be
// taken side by side: the kernels without streams have the registers for one more
// wave per SIMD (51^3, 64 columns: 72 us a product, 77 with streams).
void use_runs(cg_ctx* c, const int* found)
{
    const int fours = (c->n + kRunRows - 1) / kRunRows;
    c->streams = found[1] > 0 || 32LL * found[0] > fours;
    c->mostly_runs = 2LL * found[2] > fours;
}

RunMap<double> run_map(const cg_ctx* c) { return {c->n, c->runs, c->rowptr, c->col, c->val, nullptr}; }

// Y = A X (row-major N x s).
template <SpmmKind KIND>
__global__ __launch_bounds__(kSpmmBS, spmm_waves(KIND)) void k_spmm(RunMap<double> m, const double* __restrict__ X,
                                                  double* __restrict__ Y, int s, int G)
{
    spmm_block<KIND>(m, X, Y, s, G);
}

// A row per wave serves small matrices, whose fours of rows would leave most of the
// card idle, as long as a wave has few rows: up to 16^3 of a lattice, whose fours
// need half the gathers (64 columns, 10^3, 16^3, 20^3: 4.2, 6.5, 10.5 us against 13.9,
// 8.2, 10.6), and up to 24^3 of other rows (in random order 19 us and 21, 107 entries
// a row 61 and 63; a mesh of 20000 nodes 23 and 20), as
// to one column, for which runs save nothing (20^3 11 and 13).
static bool spmm_single(const cg_ctx* c, int s) { return c->n <= (c->mostly_runs && s > 1 ? 6144 : 16384); }

static void launch_spmm(cg_ctx* c, const double* X, double* Y, int s, int wpc)
{
    const bool single = spmm_single(c, s);
    const int G = single ? spmm_grid(c, 8, 1) : spmm_grid(c, wpc);
    const auto kernel = single ? k_spmm<SPMM_SINGLE> : c->streams ? k_spmm<SPMM_FOURS_STREAMS> : k_spmm<SPMM_FOURS>;
    kernel<<<G, kSpmmBS, 0, c->stream>>>(run_map(c), X, Y, s, G);
    JPCG_HIP(hipGetLastError());
}

// The multi-column product's grid: workgroups per CU.  Without autotune the
// default, 5, what the solver's product has registers for (51^3, 64 columns: 169
// us an iteration with 5, 173 with 4, 175 with 6, 170 with 10); with it, the first
// use times the 64-column product at 1, 2, 3, 4, 6 and 8 workgroups per CU and
// keeps the fastest.
constexpr int kSpmmDefaultWpc = 5;

int spmm_blocks_per_cu(cg_ctx* c)
{
    if (c->spmm_wpc > 0) return c->spmm_wpc;
    if (!c->opts.autotune) return c->spmm_wpc = kSpmmDefaultWpc;
    const int s = kCols;
    const size_t nb = sizeof(double) * (size_t)c->n * s;
    double *X = nullptr, *Y = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int best_w = kSpmmDefaultWpc;
    float best = 1e30f;
    try {
        JPCG_HIP(hipMalloc(&X, nb));
        JPCG_HIP(hipMalloc(&Y, nb));
        JPCG_HIP(hipMemsetAsync(X, 0, nb, c->stream));
        JPCG_HIP(hipEventCreate(&e0));
        JPCG_HIP(hipEventCreate(&e1));
        for (int w : {1, 2, 3, 4, 6, 8}) {
            launch_spmm(c, X, Y, s, w);
            JPCG_HIP(hipEventRecord(e0, c->stream));
            constexpr int kReps = 8;
            for (int r = 0; r < kReps; ++r)
                launch_spmm(c, X, Y, s, w);
            JPCG_HIP(hipEventRecord(e1, c->stream));
            JPCG_HIP(hipEventSynchronize(e1));
            float ms = 0.f;
            JPCG_HIP(hipEventElapsedTime(&ms, e0, e1));
            ms /= kReps;
            if (ms < best) {
                best = ms;
                best_w = w;
            }
        }
    } catch (...) {
        if (X) (void)hipFree(X);
        if (Y) (void)hipFree(Y);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        throw;
    }
    (void)hipFree(X);
    (void)hipFree(Y);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    c->tuned_spmm_us = best * 1e3;
    return c->spmm_wpc = best_w;
}

// Workgroups per CU of the elementwise kernels.
constexpr int kMrVectorWpc = 4;
// Blocks and matrix together from which on R and X are read and written past
// the 256 MB last-level cache, which then keeps the matrix, P and Q: at 51^3
// with 44, 48, 52 and 64 columns (268, 298, 319 and 383 MB) 146, 149, 155 and
// 169 us per iteration against 139, 149, 168 and 205 through the cache.
constexpr double kMrStreamBytes = 300e6;

template <SpmmKind KIND, typename T>
static void set_products(cg_multi* m)
{
    m->product = (const void*)k_mr_product<KIND, T>;
    m->residual = (const void*)k_mr_residual<KIND, T>;
}

template <typename T>
static cg_multi* make_multi(cg_ctx* c, int s)
{
    int wpc = spmm_blocks_per_cu(c), rows = kRunRows;
    cg_multi* m = new cg_multi();
    try {
        m->s = s;
        m->fp32 = sizeof(T) == 4;
        m->chunk = 8;
        set_products<SPMM_FOURS, T>(m);
        if (c->streams) set_products<SPMM_FOURS_STREAMS, T>(m);
        if constexpr (sizeof(T) == 4) {
            if (!c->mostly_runs) {
                set_products<SPMM_SINGLE, T>(m);
                wpc = spmm_waves(SPMM_SINGLE);
                rows = 1;
            }
        }
        const size_t ns = (size_t)c->n * s;
        m->stream = sizeof(T) * 5.0 * (double)ns + (sizeof(T) + 4.0) * (double)c->nnz > kMrStreamBytes;
        MrArgs<T>& a = margs<T>(m);
        a.G = spmm_grid(c, wpc, rows);
        a.Gv = std::max(8, std::min(c->cus * kMrVectorWpc, (c->n + 63) / 64) / 8 * 8);
        a.rows = (c->n + a.Gv - 1) / a.Gv;
        JPCG_HIP(hipMalloc(&m->work, sizeof(T) * ns * 5));
        JPCG_HIP(hipMalloc(&m->part, sizeof(double) * (size_t)std::max(a.G, a.Gv) * 3 * kWave));
        JPCG_HIP(hipMalloc(&m->st, sizeof(MrState)));
        JPCG_HIP(hipHostMalloc(&m->hst, sizeof(MrState), hipHostMallocDefault));
        JPCG_HIP(hipEventCreateWithFlags(&m->ev, hipEventDisableTiming));
        JPCG_HIP(hipMemsetAsync(m->work, 0, sizeof(T) * ns * 5, c->stream));
        JPCG_HIP(hipMemsetAsync(m->st, 0, sizeof(MrState), c->stream));
        T* w = (T*)m->work;
        a.n = c->n;
        a.s = s;
        if constexpr (sizeof(T) == 4) {
            a.m = {c->n, c->runs, c->rowptr, c->col, c->val32, c->rowsum32};
            a.dinv = c->dinv32;
        } else {
            a.m = run_map(c);
            a.dinv = c->dinv;
        }
        a.R = w;
        a.P = w + ns;
        a.Q = w + 2 * ns;
        a.B = w + 3 * ns;
        a.X = w + 4 * ns;
        a.part = m->part;
        a.st = m->st;
        a.maxit = c->n;
        a.tol = 1e-10;
        a.confirm = 1;
        JPCG_HIP(hipStreamSynchronize(c->stream));
        return m;
    } catch (...) {
        destroy_multi(m);
        throw;
    }
}

// (Re)capture the chunk graph; tol, maxit and confirm are kernel arguments.
template <typename T>
static void capture_multi(cg_multi* m)
{
    if (m->exec) (void)hipGraphExecDestroy(m->exec);
    m->exec = nullptr;
    MrArgs<T>& args = margs<T>(m);
    const bool pairs = args.s % 2 == 0;
    const void* const directions[2][2] = {
        {(const void*)k_mr_direction<1, false, T>, (const void*)k_mr_direction<1, true, T>},
        {(const void*)k_mr_direction<2, false, T>, (const void*)k_mr_direction<2, true, T>}};
    const void* const updates[2][2] = {
        {(const void*)k_mr_update<1, false, T>, (const void*)k_mr_update<1, true, T>},
        {(const void*)k_mr_update<2, false, T>, (const void*)k_mr_update<2, true, T>}};
    const void *direction = directions[pairs][m->stream], *update = updates[pairs][m->stream];
    hipStream_t cap;
    JPCG_HIP(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
    hipGraph_t graph;
    JPCG_HIP(hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal));
    for (int it = 0; it < m->chunk; ++it) {
        int ph_sig = MR_SIGMA, ph_it = MR_ITER;
        void* a0[] = {&args};
        mr_launch(direction, args.Gv, kMrBS, cap, a0);
        mr_launch(m->product, args.G, kMrBS, cap, a0);
        void* a1[] = {&args, &ph_sig};
        mr_launch((const void*)k_mr_scalars<T>, kCols, 256, cap, a1);
        mr_launch(update, args.Gv, kMrBS, cap, a0);
        void* a2[] = {&args, &ph_it};
        mr_launch((const void*)k_mr_scalars<T>, kCols, 256, cap, a2);
    }
    JPCG_HIP(hipStreamEndCapture(cap, &graph));
    hipError_t e = hipGraphInstantiate(&m->exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    JPCG_HIP(e);
    JPCG_HIP(hipStreamDestroy(cap));
}

void free_multi(cg_ctx* c)
{
    destroy_multi(c->multi);
    c->multi = nullptr;
    destroy_multi(c->multi32);
    c->multi32 = nullptr;
}

static MrState mr_read(cg_ctx* c, cg_multi* m)
{
    JPCG_HIP(hipMemcpyAsync(m->hst, m->st, sizeof(MrState), hipMemcpyDeviceToHost, c->stream));
    JPCG_HIP(hipStreamSynchronize(c->stream));
    return *m->hst;
}

// The context's multi-RHS solver of precision T for block width s, with its
// graphs captured for (tol, maxit, confirm).
template <typename T>
static cg_multi* multi_for(cg_ctx* c, int s, double tol, int maxit, int confirm)
{
    cg_multi*& slot = sizeof(T) == 4 ? c->multi32 : c->multi;
    if (!slot || slot->s != s) {
        destroy_multi(slot);
        slot = nullptr;
        slot = make_multi<T>(c, s);
    }
    MrArgs<T>& a = margs<T>(slot);
    if (!slot->exec || a.tol != tol || a.maxit != maxit || a.confirm != confirm) {
        a.tol = tol;
        a.maxit = maxit;
        a.confirm = confirm;
        capture_multi<T>(slot);
    }
    return slot;
}

// One multi-RHS solve on the solver's own B and X: setup, chunks of
// iterations, true-residual checks of waiting columns (confirm = 1), and the
// final report.  Returns the final state.
template <typename T>
static MrState run_multi(cg_ctx* c, cg_multi* m)
{
    MrArgs<T>& args = margs<T>(m);
    hipStream_t st = c->stream;
    const int s = m->s;
    int mode = 0, ph = MR_SETUP;
    void* ra[] = {&args, &mode};
    mr_launch(m->residual, args.G, kMrBS, st, ra);
    void* sa[] = {&args, &ph};
    mr_launch((const void*)k_mr_scalars<T>, kCols, 256, st, sa);
    void* za[] = {&args};
    mr_launch((const void*)k_mr_zero_cols<T>, 256, 256, st, za);
    auto flush = [&] {
        void* fa[] = {&args};
        mr_launch((const void*)k_mr_flush<T>, args.Gv, kMrBS, st, fa);
        k_mr_flushed<<<1, kCols, 0, st>>>(m->st);
        JPCG_HIP(hipGetLastError());
    };
    const long long guard = 4LL * args.maxit + 64;
    long long launched = 0;
    while (true) {
        MrState h = mr_read(c, m);
        bool active = false, pending = false;
        for (int j = 0; j < s; ++j) {
            active = active || h.status[j] == COL_ACTIVE;
            pending = pending || h.status[j] == COL_PENDING;
        }
        if (!active) {
            flush();
            if (!pending) break;
            mode = 1;
            ph = MR_CHECK;
            mr_launch(m->residual, args.G, kMrBS, st, ra);
            mr_launch((const void*)k_mr_scalars<T>, kCols, 256, st, sa);
            continue;
        }
        if (launched > guard) throw HipError{hipErrorUnknown, "multi-RHS solver did not stop"};
        // Two chunks per poll keep the device busy while the host reads.
        JPCG_HIP(hipGraphLaunch(m->exec, st));
        JPCG_HIP(hipGraphLaunch(m->exec, st));
        launched += 2 * m->chunk;
    }
    if (args.confirm) {
        mode = 2;
        ph = MR_REPORT;
        mr_launch(m->residual, args.G, kMrBS, st, ra);
        mr_launch((const void*)k_mr_scalars<T>, kCols, 256, st, sa);
    }
    return mr_read(c, m);
}

static int col_code(int status)
{
    if (status == COL_MAXIT) return CG_MAXIT;
    if (status == COL_BREAKDOWN) return CG_BREAKDOWN;
    return CG_CONVERGED;
}

}  // namespace jpcg

using namespace jpcg;

extern "C" {

int spmm(cg_ctx* c, const double* X, double* Y, int32_t s)
{
    if (!c) return CG_EINVAL;
    if (!X || !Y || X == Y || s < 1 || s > kCols) return set_error(c, CG_EINVAL, "spmm: bad arguments");
    try {
        launch_spmm(c, X, Y, s, spmm_blocks_per_cu(c));
        return 0;
    } catch (const HipError& e) {
        return set_error(c, CG_EHIP, std::string("spmm: ") + e.what + ": " + hipGetErrorString(e.code));
    }
}

int cg_solve_multi(cg_ctx* c, const double* B, double* X, int32_t s, double tol, int32_t maxit, cg_info* info)
{
    if (!c) return CG_EINVAL;
    if (!B || !X || B == X || s < 1 || s > kCols || !(tol >= 0.0) || !std::isfinite(tol))
        return set_error(c, CG_EINVAL, "cg_solve_multi: bad arguments");
    if (maxit <= 0) maxit = c->n;
    try {
        cg_multi* m = multi_for<double>(c, s, tol, maxit, 1);
        hipStream_t st = c->stream;
        const size_t nb = sizeof(double) * (size_t)c->n * s;
        JPCG_HIP(hipEventRecord(c->ev0, st));
        JPCG_HIP(hipMemcpyAsync((void*)m->args.B, B, nb, hipMemcpyDeviceToDevice, st));
        JPCG_HIP(hipMemcpyAsync(m->args.X, X, nb, hipMemcpyDeviceToDevice, st));
        const MrState h = run_multi<double>(c, m);
        JPCG_HIP(hipMemcpyAsync(X, m->args.X, nb, hipMemcpyDeviceToDevice, st));
        JPCG_HIP(hipEventRecord(c->ev1, st));
        JPCG_HIP(hipEventSynchronize(c->ev1));
        float ms = 0.f;
        JPCG_HIP(hipEventElapsedTime(&ms, c->ev0, c->ev1));
        int worst = CG_CONVERGED;
        for (int j = 0; j < s; ++j) {
            const int code = col_code(h.status[j]);
            worst = std::max(worst, code);
            if (info) {
                cg_info& o = info[j];
                o.iters = h.iters[j];
                o.status = code;
                o.replacements = h.repl[j];
                o.outer = 0;
                o.relres_recur = h.nb[j] > 0 ? std::sqrt(h.rr[j]) / h.nb[j] : 0.0;
                o.relres_true = h.nb[j] > 0 ? std::sqrt(h.rr_true[j]) / h.nb[j] : 0.0;
                o.seconds = ms * 1e-3;
            }
        }
        return worst;
    } catch (const HipError& e) {
        return set_error(c, CG_EHIP, std::string("cg_solve_multi: ") + e.what + ": " + hipGetErrorString(e.code));
    }
}

int cg_solve_multi_mixed(cg_ctx* c, const double* B, double* X, int32_t s, double tol, int32_t maxit_outer,
                         double tol_inner, int32_t maxit_inner, cg_info* info)
{
    if (!c) return CG_EINVAL;
    if (!c->val32) return set_error(c, CG_EINVAL, "cg_solve_multi_mixed: the context was created without fp32_copy");
    if (!B || !X || B == X || s < 1 || s > kCols || !(tol >= 0.0) || !std::isfinite(tol) || !(tol_inner >= 0.0) ||
        !std::isfinite(tol_inner))
        return set_error(c, CG_EINVAL, "cg_solve_multi_mixed: bad arguments");
    if (maxit_outer <= 0) maxit_outer = 50;
    if (maxit_inner <= 0) maxit_inner = c->n;
    if (tol_inner == 0.0) tol_inner = 1e-3;
    try {
        // The FP64 solver holds B, X and the outer residual (its setup phase
        // is the FP64 test); the FP32 solver runs the inner solves.
        cg_multi* m64 = multi_for<double>(c, s, tol, c->n, 1);
        cg_multi* m32 = multi_for<float>(c, s, tol_inner, maxit_inner, 0);
        hipStream_t st = c->stream;
        const size_t nb = sizeof(double) * (size_t)c->n * s;
        JPCG_HIP(hipEventRecord(c->ev0, st));
        JPCG_HIP(hipMemcpyAsync((void*)m64->args.B, B, nb, hipMemcpyDeviceToDevice, st));
        JPCG_HIP(hipMemcpyAsync(m64->args.X, X, nb, hipMemcpyDeviceToDevice, st));
        int final_status[kCols];
        int inner_iters[kCols] = {};
        for (int j = 0; j < kCols; ++j) final_status[j] = -1;
        int n = c->n;
        const int eg = std::min(4096, (c->n + 3) / 4);
        MrState h{};
        int outer = 0;
        for (;; ++outer) {
            // r = b - A x in FP64 and the per-column tests.
            int mode = 0, ph = MR_SETUP;
            void* ra[] = {&m64->args, &mode};
            mr_launch(m64->residual, m64->args.G, kMrBS, st, ra);
            void* sa[] = {&m64->args, &ph};
            mr_launch((const void*)k_mr_scalars<double>, kCols, 256, st, sa);
            if (outer == 0) {  // x_j = 0 for b_j = 0
                void* za[] = {&m64->args};
                mr_launch((const void*)k_mr_zero_cols<double>, 256, 256, st, za);
            }
            h = mr_read(c, m64);
            bool any = false, changed = false;
            for (int j = 0; j < s; ++j) {
                if (final_status[j] >= 0) {  // decided earlier: keep it out of the inner solves
                    if (h.status[j] == COL_ACTIVE) {
                        h.status[j] = final_status[j] == CG_BREAKDOWN ? COL_BREAKDOWN : COL_MAXIT;
                        changed = true;
                    }
                    continue;
                }
                if (!(h.rr[j] == h.rr[j]) || !(h.nb[j] == h.nb[j])) {  // NaN input
                    final_status[j] = CG_BREAKDOWN;
                    h.status[j] = COL_BREAKDOWN;
                    changed = true;
                } else if (h.status[j] != COL_ACTIVE) {
                    final_status[j] = CG_CONVERGED;  // converged (or b_j = 0)
                } else if (outer >= maxit_outer) {
                    final_status[j] = CG_MAXIT;
                    h.status[j] = COL_MAXIT;
                    changed = true;
                } else {
                    any = true;
                }
            }
            if (!any) break;
            if (changed) {
                int* dstatus = (int*)((char*)m64->st + offsetof(MrState, status));
                JPCG_HIP(hipMemcpyAsync(dstatus, h.status, sizeof(int) * kCols, hipMemcpyHostToDevice, st));
            }
            // Scaled residual of the active columns into the FP32 solver.
            const double* r64 = m64->args.R;
            void* ka[] = {&n, &s, &r64, &m64->st, &m32->args32.B, &m32->args32.X};
            mr_launch((const void*)k_mr_scale, eg, 256, st, ka);
            const MrState hi = run_multi<float>(c, m32);
            for (int j = 0; j < s; ++j)
                if (h.status[j] == COL_ACTIVE) inner_iters[j] += hi.iters[j];
            const float* x32 = m32->args32.X;
            void* fa[] = {&n, &s, &m64->args.X, &x32, &m64->st};
            mr_launch((const void*)k_mr_fold, eg, 256, st, fa);
        }
        JPCG_HIP(hipMemcpyAsync(X, m64->args.X, nb, hipMemcpyDeviceToDevice, st));
        JPCG_HIP(hipEventRecord(c->ev1, st));
        JPCG_HIP(hipEventSynchronize(c->ev1));
        float ms = 0.f;
        JPCG_HIP(hipEventElapsedTime(&ms, c->ev0, c->ev1));
        int worst = CG_CONVERGED;
        for (int j = 0; j < s; ++j) {
            const int code = final_status[j] < 0 ? CG_MAXIT : final_status[j];
            worst = std::max(worst, code);
            if (info) {
                cg_info& o = info[j];
                o.iters = inner_iters[j];
                o.status = code;
                o.replacements = 0;
                o.outer = outer;
                const double rel = h.nb[j] > 0 ? std::sqrt(h.rr[j]) / h.nb[j] : 0.0;
                o.relres_recur = rel;
                o.relres_true = rel;
                o.seconds = ms * 1e-3;
            }
        }
        return worst;
    } catch (const HipError& e) {
        return set_error(c, CG_EHIP,
                         std::string("cg_solve_multi_mixed: ") + e.what + ": " + hipGetErrorString(e.code));
    }
}

}  // extern "C"
