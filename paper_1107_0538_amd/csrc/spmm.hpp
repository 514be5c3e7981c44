// Row-block sparse products over row-major N x s blocks (s <= 64), shared by
// the multi-RHS and block forms.  Every column's row sum runs in stored order
// with separate multiply and add, so column j equals the sequential CSR
// product.
//
// A wave takes four rows at a time.  Rows of a structured matrix next to each
// other read runs of neighbouring columns: where the four rows' entries are
// runs of three, each row's run one column further than the row's before
// (c, c+1, c+2 in the first, c+1, c+2, c+3 in the second ...), the four rows'
// twelve entries read six rows of X, and are added from registers.  Which fours
// are such is found once per matrix (k_find_runs, a word per four rows); other
// rows of up to 32 entries are added side by side, four at a time, with a
// gather per entry, and longer ones one after the other.
//
// What bounds it: the vector-memory address path (16 clocks per instruction,
// whatever its width) and the latency of the matrix, about equally.  A gather
// therefore fetches two rows of X with 16 bytes per lane, which
// v_permlane32_swap turns into a lane per column; and four rows' values and
// columns are loaded at once, across the lanes and a step ahead, and broadcast
// by v_readlane.  Product at 51^3, 64 columns (41 MB matrix, 68 MB in, 68 MB
// out), all in the last-level cache: 204 us with a row per wave and two of the
// row's entries per gather; 121 with a row per wave in the order below and
// values through the scalar cache; 77 with four rows, 8 bytes per lane; 59 with
// 16 bytes per lane and the matrix still through the scalar cache, but 107 when
// the matrix comes from memory, one miss after the other; as it is 66, and 83
// from memory.  Rows that are not runs, 64 columns, against a row per wave with
// two entries to a gather: 51^3 in random order 239 us and 266; meshes of 20000,
// 60000 and 300000 nodes with 16 entries a row 21, 49, 241 and 26, 67, 307; rows of
// 39 (up to 66) and 107 (125) entries 47, 63 and 57, 65.  Long and unequal rows one
// after the other, 9 entries in flight, had taken 112 and 150 us, and side by side
// the meshes 34, 69 and 277.
//
// Order: the waves of one XCD walk its share of the rows side by side, so the
// rows of X between a row's first and last entry (two planes of a lattice, 2.7
// MB at 51^3) stay in that XCD's 4 MB L2 while they are needed.
#pragma once

#include <algorithm>

#include "context.hpp"

namespace jpcg {

constexpr int kRunRows = 4;   // rows of a wave's step
constexpr int kSpmmBS = 256;
constexpr int kSpmmXcds = 8;

template <typename T>
struct alignas(sizeof(T)) Pair {  // two neighbouring columns; s may be odd
    T x, y;
};

// a's upper half of the wave against b's lower half.
__device__ __forceinline__ void swap_halves(double& a, double& b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double((int)hi[0], (int)lo[0]);
    b = __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ void swap_halves(float& a, float& b)
{
    const auto w = __builtin_amdgcn_permlane32_swap(__float_as_int(a), __float_as_int(b), false, false);
    a = __int_as_float((int)w[0]);
    b = __int_as_float((int)w[1]);
}

// A lane's columns.  In pairs, lane l of either half holds columns c and c + 1
// of the half's row; in the form for sums it holds column c + half.  Lanes past
// the last column repeat it, and in a block of odd width the last pair repeats
// one column: first() and second() say which of a lane's columns are its own.
struct SpmmLane {
    int s, half, c;
    bool own1, own2;
    __device__ explicit SpmmLane(int s_) : s(s_)
    {
        const int l = threadIdx.x & 31;
        half = (threadIdx.x >> 5) & 1;
        c = s > 1 ? min(2 * l, s - 2) : 0;
        own1 = 2 * l == c && (s > 1 || half == 0);
        own2 = s > 1 && 2 * l < s;
    }
    __device__ bool own() const { return half ? own2 : own1; }  // of the form for sums
    __device__ int column() const { return s > 1 ? c + half : 0; }
    // Pairs of rows i and i + 1.
    template <typename T>
    __device__ Pair<T> load(const T* p, size_t i) const
    {
        return *(const Pair<T>*)(p + (i + half) * s + c);
    }
    template <typename T>
    __device__ void store(T* p, size_t i, T a, T b) const
    {
        T* q = p + (i + half) * s + c;
        if (own2) *(Pair<T>*)q = Pair<T>{a, b};
    }
};

template <typename T>
struct RunMap {
    int n;
    const int* __restrict__ runs;  // per four rows: entries of each if they are runs, else SPMM_EVEN or SPMM_STREAM
    const int* __restrict__ rowptr;
    const int* __restrict__ col;
    const T* __restrict__ val;
    const T* __restrict__ rowsum;  // row-sum-preserving form
};
// Fours of rows that are not runs: side by side, or as a stream.
constexpr int SPMM_EVEN = 0, SPMM_STREAM = -1;
constexpr int kSpmmShort = 32;      // longest row side by side: half a wave holds it
constexpr double kSpmmPadding = 1.25;  // entries of four rows side by side over those that they have, at most

// The kernels that a matrix's products run through: fours of rows without streams,
// which takes those that are to be streams side by side; with them; and a row per
// wave, for small matrices and, with FP32 values, all that are not mostly runs.
enum SpmmKind : int { SPMM_FOURS = 0, SPMM_FOURS_STREAMS = 1, SPMM_SINGLE = 2 };
// Waves per SIMD: what their registers allow.
constexpr int spmm_waves(SpmmKind kind) { return kind == SPMM_FOURS ? 6 : kind == SPMM_FOURS_STREAMS ? 5 : 6; }

template <bool DIFF, typename T>
__device__ __forceinline__ T spmm_add(T acc, T v, T y, T xi)
{
#pragma clang fp contract(off)
    if constexpr (DIFF) return fma_t(v, y - xi, acc);
    else return acc + v * y;
}

// A product rounded on its own, whatever it is added to.
template <typename T>
__device__ __forceinline__ T spmm_product(T v, T y)
{
#pragma clang fp contract(off)
    const T p = v * y;
    return p;
}

__device__ __forceinline__ int lane_value(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_value(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// What no kernel writes while it is read, for loads through the scalar cache.
template <typename U>
__device__ __forceinline__ auto scalar_cached(const U* p)
{
    return (const __attribute__((address_space(4))) U*)(uintptr_t)p;
}

// Four rows' values and columns across the lanes: rows 0 and 1 in the halves of
// v[0] and c[0], 2 and 3 in those of v[1] and c[1]; of a stream the first 64
// entries in v[0] and c[0], the next in v[1] and c[1].
template <typename T, bool STREAM>
struct SpmmFour {
    T v[2];
    int c[2];
    int k[kRunRows + 1];  // first entries of the rows
    int word;

    __device__ void find(const RunMap<T>& m, int g)
    {
        word = m.runs[g];
#pragma unroll
        for (int r = 0; r <= kRunRows; ++r) k[r] = m.rowptr[min(g * kRunRows + r, m.n)];
    }
    __device__ void fetch(const RunMap<T>& m)
    {
        if (STREAM && word == SPMM_STREAM) {
            part(m, k[0], 0);
            part(m, k[0] + kWave, 1);
            return;
        }
        const int l = threadIdx.x & 31;
        const bool up = (threadIdx.x & 32) != 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ka = up ? k[2 * h + 1] : k[2 * h], kb = up ? k[2 * h + 2] : k[2 * h + 1];
            v[h] = T(0);
            c[h] = 0;
            if (ka + l < kb) {
                v[h] = m.val[ka + l];
                if (h == 0 || word <= 0) c[h] = m.col[ka + l];
            }
        }
    }
    // Entries k0 to k0 + 63 of the stream (past its end: 0 in column 0).
    __device__ void part(const RunMap<T>& m, int k0, int h)
    {
        const int e = k0 + (int)(threadIdx.x & (kWave - 1));
        v[h] = T(0);
        c[h] = 0;
        if (e < k[kRunRows]) {
            v[h] = m.val[e];
            c[h] = m.col[e];
        }
    }
    __device__ T value(int r, int e) const { return lane_value(v[r / 2], 32 * (r & 1) + e); }
    __device__ int column(int r, int e) const { return lane_value(c[r / 2], 32 * (r & 1) + e); }
};

// An entry of a stream as the wave's lanes read it from LDS.
template <typename T>
struct alignas(16) SpmmEntry {
    T v;
    size_t row;  // where the column's row of X begins, in elements
};

// The six rows of X that a run of three in each of four rows reads, from the
// first one's column on.
template <typename T>
__device__ __forceinline__ void spmm_gather(const T* __restrict__ X, int s, int column, unsigned lane_at,
                                            T (&y)[kRunRows + 2])
{
    const T* p = X + (size_t)column * s;
#pragma unroll
    for (int j = 0; j < kRunRows + 2; j += 2) {
        const Pair<T> d = *(const Pair<T>*)(p + (size_t)j * s + lane_at);
        y[j] = d.x;
        y[j + 1] = d.y;
    }
}

// A X over all rows.  own(i) is asked for what the caller needs of rows i and
// i + 1 (of the half's row) while the rows' last gathers are in flight;
// two(i, u, w, o) gets rows i and i + 1 in pairs (u of the lane's first column,
// w of its second, in the half's row) with it, one(i, a) a row by itself in the
// form for sums.  DIFF: the row-sum-preserving form, sum of a_ij (x_j - x_i) +
// s_i x_i with s_i the row sum, so the near-constant modes of A are not lost to
// FP32 cancellation.
template <bool DIFF, SpmmKind KIND, typename T, typename Own, typename Two, typename One>
__device__ __forceinline__ void spmm_rows(const RunMap<T>& m, const T* __restrict__ X, const SpmmLane& L, int G,
                                          Own own, Two two, One one)
{
    constexpr int R = kRunRows, NW = kSpmmBS / kWave, B = 3;  // B: runs in flight together
    constexpr bool STREAM = KIND == SPMM_FOURS_STREAMS;
    const int s = L.s;
    const unsigned lane_at = (unsigned)(L.c + L.half * s);
    // Gathers of one value per lane take lane l column l (lanes of a half two
    // columns apart touch twice the lines); the sums change to the form for sums.
    const int column = L.column(), plain = min((int)(threadIdx.x & (kWave - 1)), s - 1);
    if constexpr (KIND == SPMM_SINGLE) {
        // Values and columns through the scalar cache, 16 gathers of 4 bytes a lane
        // in flight: FP32 values need no more (16-byte gathers and a matrix that
        // comes across the lanes take 47 us instead of 28 on a mesh of 60000 nodes
        // with 16 entries a row and 64 columns).  The last entries read past the
        // row's end, into the next row or the arrays' zero pad, and skip those slots.
        constexpr int N = 16;
        static_assert(N <= kCsrPad, "reads past a row's end must stay within the padded arrays");
        const auto val = scalar_cached(m.val);
        const auto col = scalar_cached(m.col);
        const int W = xcd_logical_block((int)blockIdx.x, G), rows = (m.n + G - 1) / G;
        const int r1 = min((W + 1) * rows, m.n);
#pragma unroll 1
        for (int i = W * rows + __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave); i < r1; i += NW) {
            {
                const int k0 = __builtin_amdgcn_readfirstlane(m.rowptr[i]);
                const int k1 = __builtin_amdgcn_readfirstlane(m.rowptr[i + 1]);
                T acc = T(0), xi = T(0);
                if constexpr (DIFF) xi = X[(size_t)i * s + plain];
#pragma unroll 1
                for (int k = k0; k < k1; k += N) {
                    T v[N], y[N];
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        v[u] = val[k + u];
                        y[u] = X[(size_t)col[k + u] * s + plain];
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        const T sum = spmm_add<DIFF>(acc, v[u], y[u], xi);
                        acc = k + u < k1 ? sum : acc;
                    }
                }
                if constexpr (DIFF) acc = fma_t(m.rowsum[i], xi, acc);
                one(i, __shfl(acc, column));
            }
        }
        return;
    }
    const int fours = (m.n + R - 1) / R, per = (fours + kSpmmXcds - 1) / kSpmmXcds, stride = G / kSpmmXcds * NW;
    const int xcd = (int)blockIdx.x % kSpmmXcds;
    const int g1 = min((xcd + 1) * per, fours);
    int g = xcd * per + __builtin_amdgcn_readfirstlane(((int)blockIdx.x / kSpmmXcds) * NW + (int)threadIdx.x / kWave);
    if (g >= g1) return;
    SpmmFour<T, STREAM> four, next;
    next.find(m, g);
    next.fetch(m);
    for (; g < g1; g += stride) {
        const int i0 = g * R;
        four = next;
        next.find(m, min(g + stride, fours - 1));
        // The next rows' entries are asked for behind this step's last
        // gathers: loads come back in the order in which they were sent, so
        // sent before they would hold the gathers back (51^3, 64 columns, matrix
        // in the last-level cache: 137 us instead of 66).
        auto ahead = [&] {
            __builtin_amdgcn_sched_barrier(0);
            next.fetch(m);
            __builtin_amdgcn_sched_barrier(0);
        };
        if (four.word > 0 && s > 1) {
            const int len = four.word;
            T acc[R] = {}, xi[R] = {};
            if constexpr (DIFF) {
#pragma unroll
                for (int r = 0; r < R; r += 2) {
                    const Pair<T> d = L.load(X, i0 + r);
                    xi[r] = d.x;
                    xi[r + 1] = d.y;
                    swap_halves(xi[r], xi[r + 1]);
                }
            }
            auto add = [&](T(&y)[R + 2], int b) {
#pragma unroll
                for (int j = 0; j < R + 2; j += 2) swap_halves(y[j], y[j + 1]);
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int j = 0; j < 3; ++j) acc[r] = spmm_add<DIFF>(acc[r], four.value(r, b + j), y[r + j], xi[r]);
            };
            int b = 0;
#pragma unroll 1
            for (; b + 3 * B < len; b += 3 * B) {
                T y[B][R + 2];
#pragma unroll
                for (int q = 0; q < B; ++q) spmm_gather(X, s, four.column(0, b + 3 * q), lane_at, y[q]);
#pragma unroll
                for (int q = 0; q < B; ++q) add(y[q], b + 3 * q);
            }
            // The last one to B runs; what the rows do not have is gathered again and not added.
            T y[B][R + 2];
#pragma unroll
            for (int q = 0; q < B; ++q) spmm_gather(X, s, four.column(0, min(b + 3 * q, len - 3)), lane_at, y[q]);
            const auto o0 = own(i0), o2 = own(i0 + 2);
            ahead();
#pragma unroll
            for (int q = 0; q < B; ++q)
                if (b + 3 * q < len) add(y[q], b + 3 * q);
            if constexpr (DIFF) {
#pragma unroll
                for (int r = 0; r < R; ++r) acc[r] = fma_t(m.rowsum[i0 + r], xi[r], acc[r]);
            }
#pragma unroll
            for (int r = 0; r < R; r += 2) swap_halves(acc[r], acc[r + 1]);
            two(i0, acc[0], acc[1], o0);
            two(i0 + 2, acc[2], acc[3], o2);
        } else if (!STREAM || four.word != SPMM_STREAM) {
            constexpr int N = 4;  // entries of each row in flight together
            T acc[R] = {}, xi[R] = {};
            int len[R], most = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                len[r] = four.k[r + 1] - four.k[r];
                most = max(most, len[r]);
                if constexpr (DIFF) xi[r] = X[(size_t)min(i0 + r, m.n - 1) * s + plain];
            }
            if (four.word > 0) four.c[1] = four.c[0] + 2;  // runs, whose later columns were not fetched
#pragma unroll 1
            for (int k = 0; k < most; k += N) {
                T y[R][N];
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int u = 0; u < N; ++u)
                        y[r][u] = X[(size_t)four.column(r, k + u) * s + plain];  // past its end: X's row 0
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int u = 0; u < N; ++u)
                        if (k + u < len[r]) acc[r] = spmm_add<DIFF>(acc[r], four.value(r, k + u), y[r][u], xi[r]);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (i0 + r >= m.n) break;
                if constexpr (DIFF) acc[r] = fma_t(m.rowsum[i0 + r], xi[r], acc[r]);
                one(i0 + r, __shfl(acc[r], column));
            }
            ahead();
        } else if constexpr (STREAM) {
            __shared__ SpmmEntry<T> stages[NW][kWave];
            SpmmEntry<T>* const stage = stages[threadIdx.x / kWave];
            // 64 entries of the stream at a time go through LDS, from where a lane
            // reads those of its half: lanes of the lower half take the even
            // entries, of the upper the odd, so that no value or column has to be
            // broadcast (with v_readlane for all of them 77 us instead of 63 at
            // 24^3 with 107 entries a row and 64 columns).  Where a row ends its sum
            // moves to the end of acc, so that after the fourth they are in order.
            constexpr int N = 8;  // entries in flight together
            static_assert(kWave % N == 0, "a part of the stream is whole steps");
            const int lane = threadIdx.x & (kWave - 1);
            T acc[R] = {}, xi[R] = {}, t = T(0);
            int end[R], open = R;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                end[r] = four.k[r + 1];
                if constexpr (DIFF) xi[r] = X[(size_t)min(i0 + r, m.n - 1) * s + column];
            }
            auto close = [&] {
                const T x0 = xi[0];
#pragma unroll
                for (int r = 0; r < R - 1; ++r) {
                    acc[r] = acc[r + 1];
                    end[r] = end[r + 1];
                    if constexpr (DIFF) xi[r] = xi[r + 1];
                }
                acc[R - 1] = t;
                end[R - 1] = -1;
                if constexpr (DIFF) xi[R - 1] = x0;
                t = T(0);
                --open;
            };
            const T* const mine = X + L.c;
            const int stop = four.k[R];
            int k = four.k[0];
            if (k == stop) ahead();
#pragma unroll 1
            while (k < stop) {
                stage[lane] = SpmmEntry<T>{four.v[0], (size_t)four.c[0] * s};
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                four.v[0] = four.v[1];
                four.c[0] = four.c[1];
                const SpmmEntry<T>* at = stage + L.half;
                const int last = min(k + kWave, stop);
                bool more = last < stop;  // another part is to be asked for, behind the first gathers
#pragma unroll 1
                for (; k < last; k += N, at += N) {
                    SpmmEntry<T> e[N / 2];
                    T y[N];
#pragma unroll
                    for (int u = 0; u < N / 2; ++u) e[u] = at[2 * u];
                    if (s > 1) {
#pragma unroll
                        for (int u = 0; u < N / 2; ++u) {
                            const Pair<T> d = *(const Pair<T>*)(mine + e[u].row);
                            y[2 * u] = d.x;
                            y[2 * u + 1] = d.y;
                        }
                    } else {
#pragma unroll
                        for (int u = 0; u < N / 2; ++u) {
                            y[2 * u] = mine[e[u].row];
                            y[2 * u + 1] = T(0);
                        }
                    }
                    if (more) four.part(m, last + kWave, 1);
                    more = false;
                    if (k + N >= stop) ahead();
                    T w[N];
#pragma unroll
                    for (int u = 0; u < N; u += 2) {
                        w[u] = w[u + 1] = e[u / 2].v;
                        if constexpr (DIFF) {
                            swap_halves(w[u], w[u + 1]);
                        } else {
                            y[u] = spmm_product(w[u], y[u]);
                            y[u + 1] = spmm_product(w[u], y[u + 1]);
                        }
                        swap_halves(y[u], y[u + 1]);
                    }
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        while (k + u == end[0]) close();
                        if constexpr (DIFF) t = fma_t(w[u], y[u] - xi[0], t);
                        else t = t + y[u];
                    }
                }
                __builtin_amdgcn_wave_barrier();  // the part has been read
            }
            while (open > 0) close();
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (i0 + r >= m.n) break;
                if constexpr (DIFF) acc[r] = fma_t(m.rowsum[i0 + r], xi[r], acc[r]);
                one(i0 + r, acc[r]);
            }
        }
    }
}

// Y = A X.
template <SpmmKind KIND, typename T>
__device__ __forceinline__ void spmm_block(const RunMap<T>& m, const T* __restrict__ X, T* __restrict__ Y, int s,
                                           int G)
{
    const SpmmLane L(s);
    spmm_rows<false, KIND>(
        m, X, L, G, [](int) { return 0; }, [&](int i, T u, T w, int) { L.store(Y, i, u, w); },
        [&](int i, T a) {
            if (L.own()) Y[(size_t)i * s + L.column()] = a;
        });
}

// Workgroups of a product over n rows at wpc per CU: a multiple of the XCDs, and
// no more than there are fours of rows (`rows` = 1: rows) for their waves.
inline int spmm_grid(const cg_ctx* c, int wpc, int rows = kRunRows)
{
    const int per = rows * (kSpmmBS / kWave);
    return std::max(kSpmmXcds, std::min(c->cus * wpc, (c->n + per - 1) / per) / kSpmmXcds * kSpmmXcds);
}

RunMap<double> run_map(const cg_ctx* c);

}  // namespace jpcg
