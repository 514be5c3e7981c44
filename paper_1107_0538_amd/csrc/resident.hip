// Host side and kernels of the resident solver (resident.hpp): which systems
// it takes, the halo lists and column slots made once per context, and the
// launch.
#include <algorithm>
#include <cstring>
#include <mutex>

#include "resident_host.hpp"

namespace jpcg {

TestHooks& test_hooks()
{
    static thread_local TestHooks h;
    return h;
}

void rs_memory()
{
    if (test_hooks().no_memory) throw HipError{hipErrorOutOfMemory, "on-chip solver"};
}

constexpr int kMaxDevices = 64;

std::mutex& resident_mutex(int device)
{
    static std::mutex m[kMaxDevices];
    return m[device >= 0 && device < kMaxDevices ? device : 0];
}

// Column slots of one workgroup's rows.  The distinct columns outside the
// workgroup's own rows (the halo) are found in a bitmap over the system's
// columns and ranked in ascending order: own column c has slot c - (first
// row), the halo column of rank h slot (own rows) + h.  Columns read from
// outside the workgroup's group are marked in `exported`.  *flag = 1 if the
// halo has more than hcap columns.
constexpr int kIndexBS = 256;

__global__ __launch_bounds__(kIndexBS) void k_rs_index(const RsIndexJob* __restrict__ jobs,
                                                       const int* __restrict__ rowptr, const int* __restrict__ col,
                                                       int hcap, int* __restrict__ hcol, int* __restrict__ hcount,
                                                       unsigned short* __restrict__ lidx, unsigned* exported,
                                                       int* flag)
{
    __shared__ unsigned bits[kRsMaxRows / 32];
    __shared__ int before[kRsMaxRows / 32];
    __shared__ int sums[kIndexBS];
    const RsIndexJob job = jobs[blockIdx.x];
    const int words = (job.n + 31) / 32, t = threadIdx.x;
    for (int w = t; w < words; w += kIndexBS) bits[w] = 0u;
    __syncthreads();
    const int ra = job.row0 + job.first, rb = ra + job.rows;
    const int k0 = rowptr[ra], k1 = rowptr[rb];
    for (int k = k0 + t; k < k1; k += kIndexBS) {
        const int c = col[k] - job.row0;
        if (c < job.first || c >= job.first + job.rows) atomicOr(&bits[c >> 5], 1u << (c & 31));
    }
    __syncthreads();
    // Exclusive prefix of the words' counts: a run of words per thread.
    const int run = (words + kIndexBS - 1) / kIndexBS;
    const int w0 = min(t * run, words), w1 = min(w0 + run, words);
    int own = 0;
    for (int w = w0; w < w1; ++w) own += __popc(bits[w]);
    sums[t] = own;
    __syncthreads();
    int base = 0;
    for (int j = 0; j < t; ++j) base += sums[j];
    int total = 0;
    for (int j = 0; j < kIndexBS; ++j) total += sums[j];
    if (total > hcap) {
        if (t == 0) *flag = 1;
        return;
    }
    int* out = hcol + (size_t)job.slot * hcap;
    for (int w = w0; w < w1; ++w) {
        before[w] = base;
        unsigned away = 0;
        for (unsigned m = bits[w]; m; m &= m - 1) {
            const int c = 32 * w + __ffs(m) - 1;
            out[base++] = c;
            if (c < job.group_first || c >= job.group_end) away |= m & -m;
        }
        if (away) atomicOr(&exported[job.bits0 + w], away);
    }
    if (t == 0) hcount[job.slot] = total;
    __syncthreads();
    for (int k = k0 + t; k < k1; k += kIndexBS) {
        const int c = col[k] - job.row0;
        int slot;
        if (c >= job.first && c < job.first + job.rows) slot = c - job.first;
        else slot = job.rows + before[c >> 5] + __popc(bits[c >> 5] & ((1u << (c & 31)) - 1u));
        lidx[k] = (unsigned short)slot;
    }
}

// Clears the exchange words (a tag of 0 is never awaited) and keeps x.
__global__ void k_rs_clear(ulonglong2* words, int64_t pairs, const double* __restrict__ x, double* __restrict__ x0,
                           int64_t n)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = t; i < pairs; i += step) words[i] = ulonglong2{0ull, 0ull};
    for (int64_t i = t; i < n; i += step) x0[i] = x[i];
}

void launch_rs_index(hipStream_t st, const RsIndexJob* jobs, int njobs, const int* rowptr, const int* col, int hcap,
                     int* hcol, int* hcount, unsigned short* lidx, unsigned* exported, int* flag)
{
    k_rs_index<<<njobs, kIndexBS, 0, st>>>(jobs, rowptr, col, hcap, hcol, hcount, lidx, exported, flag);
    JPCG_HIP(hipGetLastError());
}

void launch_rs_clear(hipStream_t st, u64* words, size_t nwords, const double* x, double* x0, int64_t n)
{
    const int64_t pairs = (int64_t)(nwords / 2);
    k_rs_clear<<<(int)std::min<int64_t>(4096, (pairs + 255) / 256), 256, 0, st>>>((ulonglong2*)words, pairs, x, x0, n);
    JPCG_HIP(hipGetLastError());
}

template <int K, int BS, int FORM>
__global__ __launch_bounds__(BS) void k_rs_solve(RsSys s, RsRun run)
{
    extern __shared__ double pl[];
    __shared__ RsLds<BS> sh;
    // Blocks are dealt to the XCDs in turn: block b belongs to group b mod 8.
    const int group = (int)blockIdx.x % kRsXcds, member = (int)blockIdx.x / kRsXcds;
    if (group >= s.groups) return;
    RsTeam<K, BS, rs_halo(BS), FORM == RS_FP32_MATRIX> team(s, run, group * s.members + member, pl, sh.red, sh.tot,
                                                            &sh.fail);
    if constexpr (FORM == RS_SINGLE) (void)team.solve_single();
    else (void)team.solve_standard();
}

template <int FORM>
static const void* rs_kernel_form(int K, int bs)
{
    if (K <= 16) {
        if (bs == 256) return (const void*)k_rs_solve<16, 256, FORM>;
        if (bs == 640) return (const void*)k_rs_solve<16, 640, FORM>;
        return (const void*)k_rs_solve<16, 1024, FORM>;
    }
    if (bs == 256) return (const void*)k_rs_solve<28, 256, FORM>;
    if (bs == 640) return (const void*)k_rs_solve<28, 640, FORM>;
    return (const void*)k_rs_solve<28, 1024, FORM>;
}

static const void* rs_kernel(int form, int K, int bs)
{
    switch (form) {
        case RS_STANDARD: return rs_kernel_form<RS_STANDARD>(K, bs);
        case RS_SINGLE: return rs_kernel_form<RS_SINGLE>(K, bs);
        default: return rs_kernel_form<RS_FP32_MATRIX>(K, bs);
    }
}

// The team for n rows: one group (one XCD) while its workgroups hold them in
// blocks of 640 threads, else all groups.  The round across XCDs costs 1.1 us
// more than the one within an XCD; 640 rows a workgroup instead of 80 cost
// about 0.3 us more per product, and blocks of 1024 threads leave 128 registers
// a thread, so that part of the row moves to LDS.
static bool rs_geometry(int n, int cus, int& groups, int& members, int& rpw)
{
    const int per_group = std::min(cus / kRsXcds, kRsGroup);
    if (per_group < 1) return false;
    auto rows = [&](int wgs) { return std::max(kRsMinRows, (((n + wgs - 1) / wgs) + 7) / 8 * 8); };
    groups = 1;
    rpw = rows(per_group);
    if (rpw > 640) {
        groups = kRsXcds;
        rpw = rows(kRsXcds * per_group);
    }
    members = std::min(per_group, (n + groups * rpw - 1) / (groups * rpw));
    return rpw <= kRsMaxWgRows;
}

void destroy_resident(cg_resident* r)
{
    if (!r) return;
    void* ptrs[] = {r->lidx, r->hcol, r->hcount, r->exported, r->words, r->x0};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    if (r->out) (void)hipHostFree(r->out);
    delete r;
}

cg_resident* make_resident(cg_ctx* c)
{
    int maxrow = 0;
    for (int i = 0; i < c->n; ++i) maxrow = std::max(maxrow, c->h_rowptr[i + 1] - c->h_rowptr[i]);
    int groups = 0, members = 0, rpw = 0;
    if (maxrow > kRsMaxRow || c->n > kRsMaxRows || !rs_geometry(c->n, c->cus, groups, members, rpw)) return nullptr;
    cg_resident* r = new cg_resident();
    RsIndexJob* djobs = nullptr;
    int* dflag = nullptr;
    try {
        rs_memory();
        r->K = maxrow <= 16 ? 16 : 28;
        r->rpw = rpw;
        r->bs = rpw <= 256 ? 256 : rpw <= 640 ? 640 : 1024;
        r->G = groups * members;
        const int hcap = rs_halo(r->bs) * (r->bs - kWave);
        std::vector<RsIndexJob> jobs(r->G);
        for (int g = 0; g < r->G; ++g) {
            const int first = std::min(g * rpw, c->n), gf = g / members * members * rpw;
            jobs[g] = RsIndexJob{0, c->n, first, std::min(rpw, c->n - first), g, gf, gf + members * rpw, 0};
        }
        JPCG_HIP(hipMalloc(&r->lidx, sizeof(unsigned short) * (c->nnz + 1)));
        JPCG_HIP(hipMalloc(&r->hcol, sizeof(int) * (size_t)r->G * hcap));
        JPCG_HIP(hipMalloc(&r->hcount, sizeof(int) * r->G));
        const size_t ebytes = sizeof(unsigned) * ((c->n + 31) / 32);
        JPCG_HIP(hipMalloc(&r->exported, ebytes));
        JPCG_HIP(hipMemsetAsync(r->exported, 0, ebytes, c->stream));
        // Exchange: two buffers of two words per row and of the sums, in whole
        // lines, and a line for the abort word.
        const size_t xw = (2 * (size_t)c->n + 15) / 16 * 16, pw = kRsSumBytes / sizeof(u64);
        r->nwords = 2 * xw + 2 * pw + 16;
        JPCG_HIP(hipMalloc(&r->words, sizeof(u64) * r->nwords));
        JPCG_HIP(hipMalloc(&r->x0, sizeof(double) * c->n));
        JPCG_HIP(hipHostMalloc(&r->out, sizeof(RsOut) * 2, hipHostMallocDefault));
        JPCG_HIP(hipMalloc(&djobs, sizeof(RsIndexJob) * r->G));
        JPCG_HIP(hipMalloc(&dflag, sizeof(int)));
        JPCG_HIP(hipMemcpyAsync(djobs, jobs.data(), sizeof(RsIndexJob) * r->G, hipMemcpyHostToDevice, c->stream));
        JPCG_HIP(hipMemsetAsync(dflag, 0, sizeof(int), c->stream));
        launch_rs_index(c->stream, djobs, r->G, c->rowptr, c->col, hcap, r->hcol, r->hcount, r->lidx, r->exported,
                        dflag);
        int flag = 0;
        std::vector<int> hcount(r->G);
        JPCG_HIP(hipMemcpyAsync(hcount.data(), r->hcount, sizeof(int) * r->G, hipMemcpyDeviceToHost, c->stream));
        JPCG_HIP(hipMemcpyAsync(&flag, dflag, sizeof(int), hipMemcpyDeviceToHost, c->stream));
        JPCG_HIP(hipStreamSynchronize(c->stream));
        (void)hipFree(djobs);
        (void)hipFree(dflag);
        djobs = nullptr;
        dflag = nullptr;
        int slots = 0;
        if (!flag) r->halo = *std::max_element(hcount.begin(), hcount.end());
        // The single-reduction form keeps more of the halo; a context of that form
        // solves in the standard one too where it has FP32 values.
        const int form = c->form == CG_FORM_SINGLE_REDUCTION && !c->val32 ? RS_SINGLE : RS_STANDARD;
        if (flag || rs_lds(form, r->K, r->bs, r->rpw, r->halo, slots) > kRsMaxLds) {
            destroy_resident(r);
            return nullptr;
        }
        RsSys& s = r->sys;
        s.row0 = 0;
        s.n = c->n;
        s.groups = groups;
        s.members = members;
        s.rpw = rpw;
        s.exported = r->exported;
        s.rowptr = c->rowptr;
        s.lidx = r->lidx;
        s.val = c->val;
        s.val32 = c->val32;
        s.rowsum = c->rowsum64;
        s.dinv = c->dinv;
        s.hcol = r->hcol;
        s.hcount = r->hcount;
        s.hcap = hcap;
        s.sums = (char*)r->words;
        s.xch = r->words + 2 * pw;
        s.xch_step = xw;
        r->abort = (unsigned*)(s.xch + 2 * xw);
        s.out = r->out;
        return r;
    } catch (...) {
        if (djobs) (void)hipFree(djobs);
        if (dflag) (void)hipFree(dflag);
        destroy_resident(r);
        if (!out_of_memory()) throw;
        return nullptr;  // the other kernels do without
    }
}

// LDS of a workgroup: the vector and what an iteration keeps of the halo, and
// (rs_tight) the columns' offsets from double `slots` on.
size_t rs_lds(int form, int K, int bs, int rows, int halo, int& slots)
{
    slots = (rows + 1 + (1 + (form == RS_SINGLE ? kRsHaloState : 1)) * halo + 1) / 2 * 2;
    return sizeof(double) * (size_t)slots + (rs_tight(bs) ? sizeof(unsigned) * (size_t)(K / 2) * bs : 0);
}

bool run_resident(cg_ctx* c, cg_resident* r, int form, const double* b, double* x, double tol, int maxit, double drop,
                  double* hist, RsOut& res)
{
    hipStream_t st = c->stream;
    RsSys s = r->sys;
    s.b = b;
    s.x = x;
    s.hist = hist;
    RsRun run{tol, drop * drop, maxit, r->abort, &r->out[1].stop, c->limit_ticks / 80, c->limit_ticks};
    if (test_hooks().wait_limit >= 0) run.limit_first = run.limit = test_hooks().wait_limit;
    const void* fn = rs_kernel(form, r->K, r->bs);
    const size_t lds = rs_lds(form, r->K, r->bs, r->rpw, r->halo, s.lds_slots);
    if (lds > kRsMaxLds || !r->retry.now()) return false;
    JPCG_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kRsMaxLds));
    void* args[] = {&s, &run};
    // One resident solve per device at a time: two of them, each partly on
    // the card, would wait for each other.
    std::lock_guard<std::mutex> lock(resident_mutex(c->device));
    r->out->stop = RS_ABORTED;
    *run.given_up = 0;
    launch_rs_clear(st, r->words, r->nwords, x, r->x0, c->n);
    const int members = std::max(1, r->sys.members - test_hooks().absent);
    JPCG_HIP(hipLaunchKernel(fn, dim3(kRsXcds * members), dim3(r->bs), args, lds, st));
    JPCG_HIP(hipStreamSynchronize(st));
    if (test_hooks().given_up) *run.given_up = 1;
    const bool ok = !*run.given_up && r->out->stop != RS_ABORTED;
    r->retry.done(ok);
    if (!ok) {
        JPCG_HIP(hipMemcpyAsync(x, r->x0, sizeof(double) * c->n, hipMemcpyDeviceToDevice, st));
        return false;
    }
    res = *r->out;
    return true;
}

}  // namespace jpcg

extern "C" void jpcg_test_on_chip(long long wait_limit, int absent, int given_up)
{
    jpcg::TestHooks& h = jpcg::test_hooks();
    h.wait_limit = wait_limit;
    h.absent = absent;
    h.given_up = given_up != 0;
}

extern "C" void jpcg_test_no_memory(int on) { jpcg::test_hooks().no_memory = on != 0; }

extern "C" int jpcg_test_solved_on_chip(const cg_ctx* c) { return c->solved < 0 ? -1 : c->solved == CG_KERNELS_ON_CHIP; }
