// Slices of a matrix (ell.hpp) made from its device CSR, and the kernels over
// them as the solver launches them.
#include <algorithm>
#include <vector>

#include "context.hpp"
#include "ell_kernels.hpp"
#include "ell_sr.hpp"

namespace jpcg {

// One wave per slice: the rows' entries side by side; *wide = 1 if a column
// lies too far from the slice's first row.  A slice's entries lie together in the
// CSR: they come in whole lines and turn in LDS (64 * width of each; read by a lane
// per row they took 1.9 ms at 128^3, 0.44 so).
static __global__ __launch_bounds__(kEllRows) void k_ell_fill(int n, int width, const int* __restrict__ rowptr,
                                                              const int* __restrict__ col,
                                                              const double* __restrict__ val,
                                                              unsigned char* __restrict__ len,
                                                              unsigned* __restrict__ col2, double* __restrict__ out,
                                                              float* __restrict__ out32, int* wide)
{
    extern __shared__ double s_val[];
    int* s_col = (int*)(s_val + kEllRows * width);
    const int s = blockIdx.x, lane = threadIdx.x, row = s * kEllRows + lane;
    const int first = rowptr[s * kEllRows], count = rowptr[min(n, (s + 1) * kEllRows)] - first;
    for (int k = lane; k < count; k += kEllRows) {
        s_val[k] = val[first + k];
        s_col[k] = col[first + k];
    }
    const int k0 = row < n ? rowptr[row] - first : 0, m = row < n ? rowptr[row + 1] - first - k0 : 0;
    const int base = s * kEllRows - kEllCol16Bias;
    if (row < n) len[row] = (unsigned char)m;
    __syncthreads();
    for (int j = 0; j < width; j += 2) {
        unsigned w = 0;
        for (int u = 0; u < 2; ++u) {
            const bool in = j + u < m;
            const int off = in ? s_col[k0 + j + u] - base : kEllCol16Bias;
            if (off < 0 || off > 0xffff) *wide = 1;
            w |= (unsigned)(off & 0xffff) << (16 * u);
            if (j + u < width) {
                const double v = in ? s_val[k0 + j + u] : 0.0;
                const size_t o = ((size_t)s * width + j + u) * kEllRows + lane;
                out[o] = v;
                if (out32) out32[o] = (float)v;
            }
        }
        col2[((size_t)s * ((width + 1) / 2) + j / 2) * kEllRows + lane] = w;
    }
}

void destroy_ell(cg_ell* e)
{
    if (!e) return;
    void* ptrs[] = {e->len, e->col2, e->val, e->val32};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    delete e;
}

// Slices pay while the padding of unequal rows stays small (at 16^3, 14 %).
constexpr double kEllMaxPadding = 1.25;
constexpr int kEllMaxRow = 64;
// Bytes of the matrix that stay in the 256 MB last-level cache: all of it if it
// fits beside the solver's five vectors, else what they and some slack leave.
// At 128^3 (557 MB) the product alone takes 98 us with 170 MB kept, 102 with
// 120, 112 with none; an iteration 145 us with 120 or 150, 147 with 170, 159
// with none and 162 with 260.
constexpr double kEllCacheBytes = 256e6, kEllCacheSlack = 20e6;
// A product by itself may alternate with products of other matrices: a third
// of the cache.  Three 128^3 matrices in turn: 118 us with 152 MB of each kept,
// 112 with 75.
constexpr double kEllSpmvBytes = 75e6;

cg_ell* make_ell(cg_ctx* c)
{
    const int n = c->n, S = (n + kEllRows - 1) / kEllRows;
    int width = 0;
    for (int i = 0; i < n; ++i) width = std::max(width, c->h_rowptr[i + 1] - c->h_rowptr[i]);
    const double padded = (double)S * width * kEllRows;
    if (c->nnz == 0 || width > kEllMaxRow || padded > 2.0e9 ||
        padded > kEllMaxPadding * (double)c->nnz + 64.0 * kEllRows)
        return nullptr;
    cg_ell* e = new cg_ell();
    int* wide = nullptr;
    try {
        const size_t entries = (size_t)S * width * kEllRows, words = (size_t)S * ((width + 1) / 2) * kEllRows;
        JPCG_HIP(hipMalloc(&e->len, n));
        JPCG_HIP(hipMalloc(&e->col2, sizeof(unsigned) * words));
        JPCG_HIP(hipMalloc(&e->val, sizeof(double) * entries));
        if (c->val32) JPCG_HIP(hipMalloc(&e->val32, sizeof(float) * entries));
        JPCG_HIP(hipMalloc(&wide, sizeof(int)));
        JPCG_HIP(hipMemsetAsync(wide, 0, sizeof(int), c->stream));
        const size_t lds = (size_t)kEllRows * width * (sizeof(double) + sizeof(int));  // 48 KB at the widest
        k_ell_fill<<<S, kEllRows, lds, c->stream>>>(n, width, c->rowptr, c->col, c->val, e->len, e->col2, e->val,
                                                    e->val32, wide);
        JPCG_HIP(hipGetLastError());
        int h = 0;
        JPCG_HIP(hipMemcpyAsync(&h, wide, sizeof(int), hipMemcpyDeviceToHost, c->stream));
        JPCG_HIP(hipStreamSynchronize(c->stream));
        (void)hipFree(wide);
        wide = nullptr;
        if (h) {
            destroy_ell(e);
            return nullptr;
        }
        auto keep = [&](double value_bytes) {
            const double bytes = padded * (value_bytes + 2.0), room = kEllCacheBytes - 40.0 * n;
            if (bytes <= room) return 128;
            return (int)std::min(128.0, 128.0 * std::max(0.0, room - kEllCacheSlack) / bytes);
        };
        e->map = EllMap{n, S, width, e->len, e->col2, e->val, e->val32};
        e->keep = keep(8.0);
        e->keep32 = keep(4.0);
        e->keep_spmv = (int)std::min(128.0, 128.0 * kEllSpmvBytes / (padded * 10.0));
        return e;
    } catch (const HipError& err) {
        if (wide) (void)hipFree(wide);
        destroy_ell(e);
        if (err.code != hipErrorOutOfMemory) throw;
        (void)hipGetLastError();
        return nullptr;  // no room for a second copy of the matrix: the tiles do without
    }
}

// Entries in flight: 14 for rows that short, else 28.
template <int U>
static EllKernels ell_kernels_of(bool mat32)
{
    EllKernels k{};
    k.setup = (const void*)k_ell_setup<U>;
    k.begin = (const void*)k_ell_begin;
    k.direction = (const void*)k_ell_direction;
    k.product = mat32 ? (const void*)k_ell_product<true, U> : (const void*)k_ell_product<false, U>;
    k.update = (const void*)k_ell_update;
    k.flush = (const void*)k_ell_flush;
    k.flushed = (const void*)k_ell_flushed;
    k.check = (const void*)k_ell_check<U>;
    k.decide = (const void*)k_ell_decide;
    k.sr_residual = (const void*)k_ell_sr_residual<U>;
    k.sr_begin = (const void*)k_ell_sr_begin;
    k.sr_start = (const void*)k_ell_sr_start<U>;
    k.sr_update = (const void*)k_ell_sr_update;
    k.sr_product = (const void*)k_ell_sr_product<U>;
    k.sr_decide = (const void*)k_ell_sr_decide;
    return k;
}

EllKernels ell_kernels(const cg_ell* e, bool mat32)
{
    return e->map.width <= 14 ? ell_kernels_of<14>(mat32) : ell_kernels_of<28>(mat32);
}

void launch_ell_spmv(const cg_ell* e, hipStream_t st, const double* x, double* y)
{
    int G = (e->map.S + 7) / 8 * 8, keep = e->keep_spmv;
    EllMap m = e->map;
    void* args[] = {&m, &keep, &G, &x, &y};
    const void* fn = m.width <= 14 ? (const void*)k_ell_spmv<14> : (const void*)k_ell_spmv<28>;
    JPCG_HIP(hipLaunchKernel(fn, dim3(G), dim3(kEllRows), args, 0, st));
}

}  // namespace jpcg
