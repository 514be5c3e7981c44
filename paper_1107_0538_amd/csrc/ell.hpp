// Sparse products over slices of 64 rows (one wave, a lane per row), for
// matrices whose rows are about equally long.
//
// A slice stores its rows' j-th entries side by side: values [j][64], and the
// columns as 16-bit offsets from the slice's first row, two entries to a
// 32-bit word [j / 2][64], j up to the longest row of the matrix, so that a
// slice's place needs no look-up (which put a dependent load before all
// others: 10.5 us for the product at 51^3 against 9.9).  A lane adds its own
// row's products in stored order from separately rounded products, so y = A x
// is bitwise the sequential CSR product; slots past a row's end are loaded (an
// entry of the slice) and not added.
//
// What bounds it: memory.  Every load of values and columns is a full line and
// independent of the others, and neighbouring rows gather neighbouring
// columns, so a gather touches 4-5 lines where the tile walk of tiles.hpp
// (lanes along a row) touches 20 or more, and the row sums need no LDS.
// Product at 128^3 (710.9 MB in CSR, 602 MB here): 149 us by tiles, 108 here again
// and again, 112 with three matrices in turn; at 51^3 9.4 and 8.7, a launch
// included.
//
// A matrix larger than the 256 MB last-level cache is read with non-temporal
// loads except for a fixed share of its slices, spread evenly, which then stay
// in the cache from one product to the next: the product at 128^3 by itself 122 us
// with plain loads only, 112 with non-temporal ones only, 98 with 170 MB (30 %) of
// the slices kept; ell.hip says how much the solver and spmv keep.
#pragma once

#include "common.hpp"

namespace jpcg {

constexpr int kEllRows = 64;
constexpr int kEllCol16Bias = 32768;

struct EllMap {
    int n, S;                  // rows, slices
    int width;                 // entries of the longest row, and so of every slice's rows
    const unsigned char* len;  // per row: entries
    const unsigned* col2;
    const double* val;
    const float* val32;        // FP32-matrix form
};
// Slices of 128 that stay cached are an argument of their own (128: all).

template <bool STREAM, typename T>
__device__ __forceinline__ T ell_load(const T* p)
{
    if constexpr (STREAM) return __builtin_nontemporal_load(p);
    else return *p;
}

// Row `64 s + lane` of slice s: the sum over its entries, in stored order, of
// value * x[column].  With DIFF the row-sum-preserving form (see tiles.hpp):
// the sum of value * (x[column] - xi).  U: entries of a row in flight together
// (all of a 27-entry row: a second chunk's loads would wait for the first's
// gathers, 10.3 us against 9.9 at 51^3).
template <bool DIFF, int U, typename VT>
__device__ __forceinline__ double ell_row(const EllMap& m, const VT* __restrict__ vals, int keep, int s, int lane,
                                          const double* __restrict__ x, double xi)
{
#pragma clang fp contract(off)
    const int len = m.width;
    const VT* __restrict__ v = vals + (size_t)s * len * kEllRows + lane;
    const unsigned* __restrict__ c = m.col2 + (size_t)s * ((len + 1) / 2) * kEllRows + lane;
    const int row = s * kEllRows + lane;
    const int mine = row < m.n ? (int)m.len[row] : 0;
    const int base = s * kEllRows - kEllCol16Bias, self = min(row, m.n - 1);
    const bool kept = ((s * 37) & 127) < keep;
    double t = 0.0;
    for (int g = 0; g < len; g += U) {
        VT e[U];
        unsigned w[U / 2];
        const int last = len - 1;
        if (kept) {
            asm volatile("; cached");
#pragma unroll
            for (int j = 0; j < U / 2; ++j) w[j] = ell_load<false>(c + min(g + 2 * j, last) / 2 * kEllRows);
#pragma unroll
            for (int j = 0; j < U; ++j) e[j] = ell_load<false>(v + min(g + j, last) * kEllRows);
            asm volatile("; cached loads end");
        } else {
            asm volatile("; streamed");
#pragma unroll
            for (int j = 0; j < U / 2; ++j) w[j] = ell_load<true>(c + min(g + 2 * j, last) / 2 * kEllRows);
#pragma unroll
            for (int j = 0; j < U; ++j) e[j] = ell_load<true>(v + min(g + j, last) * kEllRows);
            asm volatile("; streamed loads end");
        }
        double y[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int o = (j & 1) ? (int)(w[j / 2] >> 16) : (int)(w[j / 2] & 0xffffu);
            y[j] = x[g + j < mine ? base + o : self];
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            if constexpr (DIFF) {
                const double d = __builtin_fma((double)e[j], y[j] - xi, t);
                t = g + j < mine ? d : t;
            } else {
                const double p = (double)e[j] * y[j];
                t = g + j < mine ? t + p : t;
            }
        }
    }
    return t;
}

}  // namespace jpcg
