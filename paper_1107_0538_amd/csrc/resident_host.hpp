// The resident solver as the entry points see it (resident.hip).
#pragma once

#include <mutex>

#include "context.hpp"
#include "resident.hpp"

namespace jpcg {

enum RsForm : int { RS_STANDARD = 0, RS_SINGLE = 1, RS_FP32_MATRIX = 2 };

constexpr int kRsMaxRow = 28;         // nonzeros of a row at most
constexpr int kRsMaxWgRows = 1024;    // rows of a workgroup at most
// Halo columns per thread at most.
constexpr int rs_halo(int bs) { return bs == 256 ? 4 : 3; }
// Dynamic LDS of a workgroup at most (160 KB less the kernels' static 10.3 KB).
constexpr size_t kRsMaxLds = 149 * 1024;
constexpr int kRsMinRows = 64;        // rows of a workgroup at least
constexpr int kRsMaxRows = kRsGroups * kRsGroup * kRsMaxWgRows;  // rows of a system at most (bitmap of the index kernel)

// Rows [first, first + rows) of the system with rows [row0, row0 + n): one
// workgroup's share, whose halo list goes to entry `slot`.
struct RsIndexJob {
    int row0, n, first, rows, slot;
    int group_first, group_end;  // rows of the workgroup's group
    int bits0;                   // first word of the system's `exported` bits
};

// Held by every launch whose workgroups wait for each other, until it ends.
std::mutex& resident_mutex(int device);

}  // namespace jpcg

struct cg_resident {
    int K = 0, bs = 0, G = 0, rpw = 0, halo = 0;
    size_t nwords = 0;
    unsigned short* lidx = nullptr;
    int* hcol = nullptr;
    int* hcount = nullptr;
    unsigned* exported = nullptr;
    jpcg::u64* words = nullptr;  // exchange buffers and the abort word
    unsigned* abort = nullptr;
    jpcg::RsOut* out = nullptr;  // pinned
    jpcg::RsSys sys{};
};

namespace jpcg {

// Null when the system does not fit (rows too long, too many, or referring to
// too many other rows).
cg_resident* make_resident(cg_ctx* c);
void destroy_resident(cg_resident* r);

// False if the workgroups could not all be on the card in time; x is then as
// it was.
bool run_resident(cg_ctx* c, cg_resident* r, int form, const double* b, double* x, double tol, int maxit, double drop,
                  double* hist, RsOut& res);

}  // namespace jpcg
