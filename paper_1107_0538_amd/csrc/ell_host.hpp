// Slices of a context's matrix and the kernels over them (ell.hip).
#pragma once

#include "context.hpp"
#include "ell.hpp"
#include "sr_kernels.hpp"
#include "std_kernels.hpp"

struct cg_ell {
    unsigned char* len = nullptr;
    unsigned* col2 = nullptr;
    double* val = nullptr;
    float* val32 = nullptr;
    int keep = 0, keep32 = 0, keep_spmv = 0;  // slices of 128 that stay cached: solver, FP32 values, spmv
    jpcg::EllMap map{};
};

namespace jpcg {

struct EllState {
    CgState cg;
    int pend[2];  // pend[k % 2]: x += alpha_k p_k is still to be done (set by the update)
};

struct EllArgs {
    EllMap m;
    int keep;  // slices of 128 that stay cached
    const double* __restrict__ dinv;
    const double* __restrict__ rowsum;  // FP32-matrix form
    const double* b;
    double* x;
    double* r;
    double* p;
    double* q;
    int G;    // workgroups of the product kernels
    int Gu;   // of the elementwise kernels
    int R;    // rows per workgroup of the elementwise kernels
    double* part_setup;    // [G][3]: r'r, r'z, b'b
    double* part_sig;      // [G][1]
    double* part_iter;     // [Gu][2]
    double* part_chk;      // [G][2]
    EllState* st;
    double* hist;
    double drop2;
};

// The single-reduction form (ell_sr.hpp).
struct EllSrArgs {
    EllMap m;
    int keep;
    const double* __restrict__ dinv;
    const double* b;
    double* x;
    double *r, *p, *s, *w, *u;
    int G, Gu, R;        // as above
    double* part[2];     // [Gu][4], by parity
    double* part_w;      // [G][2]
    double* part_chk;    // [G][2]
    SrState* st;
    double* hist;
};

constexpr int kEllBS = 256;
constexpr int kEllWaves = kEllBS / kWave;

struct EllKernels {
    const void *setup, *begin, *direction, *product, *update, *flush, *flushed, *check, *decide;
    const void *sr_residual, *sr_begin, *sr_start, *sr_update, *sr_product, *sr_decide;
};
EllKernels ell_kernels(const cg_ell* e, bool mat32);

// Null where slices do not suit the matrix: rows too unequal or too long, or
// columns too far from the diagonal.
cg_ell* make_ell(cg_ctx* c);
void destroy_ell(cg_ell* e);
void launch_ell_spmv(const cg_ell* e, hipStream_t st, const double* x, double* y);

}  // namespace jpcg
