// The resident solver as the entry points see it (resident.hip).
#pragma once

#include <mutex>

#include "context.hpp"
#include "resident.hpp"
#include "test_hooks.hpp"

namespace jpcg {

enum RsForm : int { RS_STANDARD = 0, RS_SINGLE = 1, RS_FP32_MATRIX = 2 };

constexpr int kRsMaxRow = 28;         // nonzeros of a row at most
constexpr int kRsMaxWgRows = 1024;    // rows of a workgroup at most
// Halo columns per thread at most.
constexpr int rs_halo(int bs) { return bs == 256 ? 4 : 3; }
// Dynamic LDS of a workgroup at most (160 KB less the kernels' static 10.3 KB).
constexpr size_t kRsMaxLds = 149 * 1024;
constexpr int kRsMinRows = 64;        // rows of a workgroup at least
constexpr int kRsMaxRows = kRsXcds * kRsGroup * kRsMaxWgRows;  // rows of a system at most (bitmap of the index kernel)

// Rows [first, first + rows) of the system with rows [row0, row0 + n): one
// workgroup's share, whose halo list goes to entry `slot`.
struct RsIndexJob {
    int row0, n, first, rows, slot;
    int group_first, group_end;  // rows of the workgroup's group
    int bits0;                   // first word of the system's `exported` bits
};

template <int BS>
struct RsLds {
    double red[kRsSums * BS / 4];
    double tot[kRsSums];
    int fail;
};

void launch_rs_index(hipStream_t st, const RsIndexJob* jobs, int njobs, const int* rowptr, const int* col, int hcap,
                     int* hcol, int* hcount, unsigned short* lidx, unsigned* exported, int* flag);
// Clears the words and copies n entries of x to x0 (n may be 0).
void launch_rs_clear(hipStream_t st, u64* words, size_t nwords, const double* x, double* x0, int64_t n);
size_t rs_lds(int form, int K, int bs, int rows, int halo, int& slots);

// Throws out of memory where a test asks for that.
void rs_memory();

// Held by every launch whose workgroups wait for each other, until it ends.
std::mutex& resident_mutex(int device);

}  // namespace jpcg

namespace jpcg {

// After a launch that was given up the next ones go to the general kernels at
// once, as the wait was in vain and what kept the workgroups off the card (other
// work, a mask of compute units) may last: one solve, then two, four and so on
// to 64, until one succeeds.
struct RsRetry {
    int skip = 0, pause = 0;
    bool now()
    {
        if (skip == 0) return true;
        --skip;
        return false;
    }
    void done(bool ok)
    {
        pause = ok ? 0 : pause == 0 ? 1 : pause < 64 ? 2 * pause : 64;
        skip = pause;
    }
};

}  // namespace jpcg

struct cg_resident {
    jpcg::RsRetry retry;
    int K = 0, bs = 0, G = 0, rpw = 0, halo = 0;
    size_t nwords = 0;
    unsigned short* lidx = nullptr;
    int* hcol = nullptr;
    int* hcount = nullptr;
    unsigned* exported = nullptr;
    jpcg::u64* words = nullptr;  // exchange buffers and the abort word
    unsigned* abort = nullptr;
    double* x0 = nullptr;        // x as the caller passed it
    jpcg::RsOut* out = nullptr;  // pinned; out[1].stop: a workgroup gave up
    jpcg::RsSys sys{};
};

namespace jpcg {

// Null when the system does not fit (rows too long, too many, or referring to
// too many other rows), or there is no memory for it.
cg_resident* make_resident(cg_ctx* c);
void destroy_resident(cg_resident* r);

// False if some workgroup gave up waiting, as when they could not all be on the
// card in time, or just after such a launch; x is then what it was.
bool run_resident(cg_ctx* c, cg_resident* r, int form, const double* b, double* x, double tol, int maxit, double drop,
                  double* hist, RsOut& res);

// The batch's systems by teams of the same solver (resident_batch.hip).
struct RsBatchMatrix {
    int nsys;
    const int* rows;         // per system
    const int64_t* row_off;  // per system, and the total
    const int* h_rowptr;     // of the concatenated matrix, on the host and the device
    const int* rowptr;
    const int* col;
    const double* val;
    const double* dinv;
};
struct cg_batch_resident;
// Null when some system does not fit, or there is no memory.
cg_batch_resident* make_batch_resident(const RsBatchMatrix& m, int cus, hipStream_t st);
void destroy_batch_resident(cg_batch_resident* r);
// Solves on the batch's own b and x (maxit <= 0: each system's rows) and fills
// out[nsys].  limit: 8 s in device ticks, the most that a round takes.  False if
// some workgroup gave up waiting, or just after such a launch: none of x counts
// then.
bool run_batch_resident(cg_batch_resident* r, int device, hipStream_t st, const double* b, double* x, double tol,
                        int maxit, long long limit, const RsOut*& out);

}  // namespace jpcg
