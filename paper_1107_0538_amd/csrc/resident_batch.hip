// Batched solves on chip: many systems, each by a team of workgroups as in
// resident.hpp, in one launch that fills the card once.
//
// A system takes as few workgroups as hold its rows, in groups of at most 32
// that sit on one XCD each.  The host deals the systems, the most
// expensive first, to the workgroup slots that come free first; each
// workgroup works through its list.  All lists follow one order of the
// systems, so the first unfinished system of that order always has its whole
// team on it and the launch makes progress.  A gate at the start of the
// kernel checks that every workgroup is on the card.
//
// Each matrix is read once per solve instead of once per iteration.  96
// systems of 12^3 to 48^3 unknowns: 170 ms with the matrices streamed by teams
// of phases.hpp, 40.9 ms here, of which the workgroups solve 89 %, wait for
// their teams 8 % and idle 3 %; 5.9 us an iteration at 42^3 to 48^3 (two such
// systems at a time), 3.5 us below 25^3.  The rounds' latency bounds it.
#include <algorithm>
#include <cmath>
#include <vector>

#include "resident_host.hpp"

namespace jpcg {

// A system's part of a launch, as 32-bit words that every lane reads alike.
struct RsBatchSys {
    int row0, n, groups, members, rpw;
    int slot0;   // first entry of its halo lists
    int bits0;   // first word of its exported bits
    int line0;   // first 128-byte line of its exchanged vectors
    int sums0;   // of its sums
};
struct RsBatchJob {
    int sys, index;  // member `index` of the system's team
};

struct RsBatchArgs {
    const RsBatchSys* sys;
    const RsBatchJob* jobs;
    const int* job_off;  // per workgroup, and the end
    RsSys common;        // bases of all systems' arrays
    RsOut* out;
    unsigned* gate;
    long long gate_limit;
    RsRun run;
};

__device__ __forceinline__ int rs_scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <int K, int BS, int NH>
__global__ __launch_bounds__(BS, BS == 512 ? 4 : 1) void k_rs_batch(RsBatchArgs a)
{
    extern __shared__ double pl[];
    __shared__ RsLds<BS> sh;
    // The gate: every workgroup arrives, or everyone leaves.
    if (threadIdx.x == 0) {
        sh.fail = 0;
        __hip_atomic_fetch_add(a.gate, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        RsWait wait(a.run, a.gate_limit);
        while (__hip_atomic_load(a.gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < gridDim.x) {
            __builtin_amdgcn_s_sleep(2);
            if (!wait.more()) {
                sh.fail = 1;
                break;
            }
        }
    }
    __syncthreads();
    if (rs_scalar(sh.fail)) return;
    // Blocks are dealt to the XCDs in turn; the lists are by XCD and slot.
    const int wg = ((int)blockIdx.x % kRsXcds) * ((int)gridDim.x / kRsXcds) + (int)blockIdx.x / kRsXcds;
    const int j1 = rs_scalar(a.job_off[wg + 1]);
    for (int j = rs_scalar(a.job_off[wg]); j < j1; ++j) {
        const int sys = rs_scalar(a.jobs[j].sys), index = rs_scalar(a.jobs[j].index);
        const RsBatchSys& t = a.sys[sys];
        RsSys s = a.common;
        s.row0 = rs_scalar(t.row0);
        s.n = rs_scalar(t.n);
        s.groups = rs_scalar(t.groups);
        s.members = rs_scalar(t.members);
        s.rpw = rs_scalar(t.rpw);
        const int slot0 = rs_scalar(t.slot0);
        s.hcol += (size_t)slot0 * s.hcap;
        s.hcount += slot0;
        s.exported += rs_scalar(t.bits0);
        s.xch += 16 * (size_t)rs_scalar(t.line0);
        s.sums += 128 * (size_t)rs_scalar(t.sums0);
        s.out = a.out + sys;
        RsRun run = a.run;
        if (run.maxit <= 0) run.maxit = s.n;
        RsTeam<K, BS, NH, false> team(s, run, index, pl, sh.red, sh.tot, &sh.fail);
        if (!team.solve_standard()) return;
        __syncthreads();  // the next system reuses the LDS
    }
}

// Halo columns per thread: of a block of 512 threads three, as far as that goes
// (rows of a 27-point lattice up to 53^3: 1332 columns for 512 rows; 128 registers
// are short, and a fourth entry makes 26 of them spill, not 20); 54^3 to 64^3 have
// up to 1408.
constexpr int kBatchHalo = 3, kBatchHaloMost = 4;
static_assert(rs_halo(256) == kBatchHaloMost, "one capacity for either block");

template <int K>
static const void* rs_batch_kernel_of(int bs, int nh)
{
    if (bs == 256) return (const void*)k_rs_batch<K, 256, rs_halo(256)>;
    if (nh == kBatchHalo) return (const void*)k_rs_batch<K, 512, kBatchHalo>;
    return (const void*)k_rs_batch<K, 512, kBatchHaloMost>;
}
static const void* rs_batch_kernel(int K, int bs, int nh)
{
    return K <= 16 ? rs_batch_kernel_of<16>(bs, nh) : rs_batch_kernel_of<28>(bs, nh);
}

struct cg_batch_resident {
    RsRetry retry;
    int nsys = 0, K = 0, bs = 0, nh = 0, grid = 0;
    size_t lds = 0, nwords = 0;
    long long rows = 0;  // of all systems
    RsBatchSys* sys = nullptr;
    RsBatchJob* jobs = nullptr;
    int* job_off = nullptr;
    unsigned short* lidx = nullptr;
    int* hcol = nullptr;
    int* hcount = nullptr;
    unsigned* exported = nullptr;
    u64* words = nullptr;
    RsOut* out = nullptr;  // pinned; behind the systems' the word of workgroups that gave up
    RsBatchArgs args{};
};

void destroy_batch_resident(cg_batch_resident* r)
{
    if (!r) return;
    void* ptrs[] = {r->sys, r->jobs, r->job_off, r->lidx, r->hcol, r->hcount, r->exported, r->words};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    if (r->out) (void)hipHostFree(r->out);
    delete r;
}

// The order of the systems and their teams' places: the most expensive first,
// each to the XCDs and slots that come free first.  jobs[wg] lists (system,
// team member) in that order.
static void rs_schedule(const std::vector<RsBatchSys>& sys, int slots, std::vector<std::vector<RsBatchJob>>& jobs)
{
    const int nsys = (int)sys.size();
    std::vector<double> cost(nsys);
    std::vector<int> order(nsys);
    for (int s = 0; s < nsys; ++s) {
        order[s] = s;
        // Iterations grow with the edge of a grid; microseconds of an
        // iteration within one XCD and across several, and of its rows.
        cost[s] = std::cbrt((double)sys[s].n) *
                  ((sys[s].groups * sys[s].members == 1 ? 1.0 : sys[s].groups == 1 ? 2.4 : 4.0) + sys[s].rpw / 500.0);
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        const double ca = cost[a] * sys[a].groups * sys[a].members, cb = cost[b] * sys[b].groups * sys[b].members;
        return ca > cb;
    });
    std::vector<std::vector<double>> free_at(kRsXcds, std::vector<double>(slots, 0.0));
    jobs.assign((size_t)kRsXcds * slots, {});
    for (int s : order) {
        const int m = sys[s].members, g = sys[s].groups;
        // Each group to the XCD that first has m more slots free.
        std::vector<int> groups_on(kRsXcds, 0);
        double start = 0.0;
        for (int k = 0; k < g; ++k) {
            int best = -1;
            double at = 0.0;
            for (int x = 0; x < kRsXcds; ++x) {
                const int need = m * (groups_on[x] + 1);
                if (need > slots) continue;
                std::vector<double> f = free_at[x];
                std::nth_element(f.begin(), f.begin() + (need - 1), f.end());
                if (best < 0 || f[need - 1] < at) {
                    best = x;
                    at = f[need - 1];
                }
            }
            groups_on[best] += 1;
            start = std::max(start, at);
        }
        int k = 0;
        for (int x = 0; x < kRsXcds; ++x) {
            if (!groups_on[x]) continue;
            std::vector<int> by(slots);
            for (int i = 0; i < slots; ++i) by[i] = i;
            // Of the slots free by then, those that have waited least.
            std::stable_sort(by.begin(), by.end(), [&](int a, int b) {
                const bool fa = free_at[x][a] <= start, fb = free_at[x][b] <= start;
                if (fa != fb) return fa;
                return fa ? free_at[x][a] > free_at[x][b] : free_at[x][a] < free_at[x][b];
            });
            for (int i = 0; i < m * groups_on[x]; ++i) {
                free_at[x][by[i]] = start + cost[s];
                jobs[(size_t)x * slots + by[i]].push_back(RsBatchJob{s, (k + i / m) * m + i % m});
            }
            k += groups_on[x];
        }
    }
}

cg_batch_resident* make_batch_resident(const RsBatchMatrix& m, int cus, hipStream_t st)
{
    const int per_xcd = std::min(cus / kRsXcds, kRsGroup);  // compute units
    if (per_xcd < 1) return nullptr;
    const int64_t total = m.row_off[m.nsys], nnz = m.h_rowptr[total];
    int maxrow = 0;
    for (int64_t i = 0; i < total; ++i) maxrow = std::max(maxrow, m.h_rowptr[i + 1] - m.h_rowptr[i]);
    if (maxrow > kRsMaxRow) return nullptr;
    // Where the batch needs the card more than once over, workgroups of 512
    // rows, two to a compute unit, so that one computes while the other waits
    // for its team (40.9 ms on the 96 systems; 42.4 with one of 1024 rows).  A
    // smaller batch is spread over all compute units.
    auto round8 = [](int64_t v) { return (int)((v + 7) / 8 * 8); };
    const int spread = round8(total / (kRsXcds * per_xcd) + 1);
    const int per_cu = spread <= 256 ? 1 : 2;
    const int slots = per_xcd * per_cu, target = per_cu == 1 ? std::max(128, spread) : 512;
    std::vector<RsBatchSys> sys(m.nsys);
    // Sums: 2 kRsSumBytes for a team of several groups; teams of one group have the
    // places of a group each, 16 to as many bytes; a workgroup alone has none.  (A
    // layout of 5 KB for a team of one group took solves of 4096 rows from 398 us to
    // 418: it matters to the caches where the two parities lie.)
    constexpr int kSumLines = (int)(2 * kRsSumBytes / 128), kGroupLines = 16 * kRsSums * kRsGroup / 128;
    int slot = 0, bits = 0, line = 0, sums = 0, shared = 0, in_shared = kRsGroups, rows_max = 0;
    for (int s = 0; s < m.nsys; ++s) {
        RsBatchSys& t = sys[s];
        const int n = m.rows[s];
        if (n > kRsMaxRows) return nullptr;
        const int wgs = (n + target - 1) / target;
        const int width = std::min(slots, kRsGroup);
        t.groups = (wgs + width - 1) / width;
        t.members = (wgs + t.groups - 1) / t.groups;
        const int teams = t.groups * t.members;
        if (teams > kRsXcds * slots || t.groups > (slots / t.members) * kRsXcds || t.groups > kRsGroups) return nullptr;
        t.rpw = std::max(8, round8((n + teams - 1) / teams));
        if (t.rpw > (per_cu == 1 ? 256 : 512)) return nullptr;
        t.row0 = (int)m.row_off[s];
        t.n = n;
        t.slot0 = slot;
        t.bits0 = bits;
        t.line0 = line;
        t.sums0 = 0;
        if (t.groups > 1) {
            t.sums0 = sums;
            sums += kSumLines;
        } else if (teams > 1) {
            if (in_shared == kRsGroups) {
                shared = sums;
                sums += kSumLines;
                in_shared = 0;
            }
            t.sums0 = shared + kGroupLines * in_shared++;
        }
        slot += teams;
        bits += (n + 31) / 32;
        line += (n + 7) / 8;
        rows_max = std::max(rows_max, t.rpw);
    }
    cg_batch_resident* r = new cg_batch_resident();
    RsIndexJob* djobs = nullptr;
    int* dflag = nullptr;
    try {
        rs_memory();
        r->nsys = m.nsys;
        r->rows = total;
        r->K = maxrow <= 16 ? 16 : 28;
        r->bs = per_cu == 1 ? 256 : 512;
        r->grid = kRsXcds * slots;
        const int hcap = kBatchHaloMost * (r->bs - kWave);
        std::vector<RsIndexJob> index(slot);
        for (const RsBatchSys& t : sys)
            for (int g = 0; g < t.groups * t.members; ++g) {
                const int first = std::min(g * t.rpw, t.n), gf = g / t.members * t.members * t.rpw;
                index[t.slot0 + g] = RsIndexJob{t.row0,       t.n, first, std::min(t.rpw, t.n - first),
                                                t.slot0 + g, gf,  gf + t.members * t.rpw, t.bits0};
            }
        std::vector<std::vector<RsBatchJob>> lists;
        rs_schedule(sys, slots, lists);
        std::vector<RsBatchJob> jobs;
        std::vector<int> job_off(1, 0);
        for (const auto& l : lists) {
            jobs.insert(jobs.end(), l.begin(), l.end());
            job_off.push_back((int)jobs.size());
        }
        const size_t xw = 16 * (size_t)line, sw = 16 * (size_t)sums;
        r->nwords = 2 * xw + sw + 32;  // a line each for the abort word and the gate
        JPCG_HIP(hipMalloc(&r->sys, sizeof(RsBatchSys) * m.nsys));
        JPCG_HIP(hipMalloc(&r->jobs, sizeof(RsBatchJob) * jobs.size()));
        JPCG_HIP(hipMalloc(&r->job_off, sizeof(int) * job_off.size()));
        JPCG_HIP(hipMalloc(&r->lidx, sizeof(unsigned short) * (nnz + 1)));
        JPCG_HIP(hipMalloc(&r->hcol, sizeof(int) * (size_t)slot * hcap));
        JPCG_HIP(hipMalloc(&r->hcount, sizeof(int) * slot));
        JPCG_HIP(hipMalloc(&r->exported, sizeof(unsigned) * bits));
        JPCG_HIP(hipMalloc(&r->words, sizeof(u64) * r->nwords));
        JPCG_HIP(hipHostMalloc(&r->out, sizeof(RsOut) * (m.nsys + 1), hipHostMallocDefault));
        JPCG_HIP(hipMalloc(&djobs, sizeof(RsIndexJob) * slot));
        JPCG_HIP(hipMalloc(&dflag, sizeof(int)));
        auto up = [&](void* d, const void* h, size_t bytes) {
            JPCG_HIP(hipMemcpyAsync(d, h, bytes, hipMemcpyHostToDevice, st));
        };
        up(r->sys, sys.data(), sizeof(RsBatchSys) * m.nsys);
        up(r->jobs, jobs.data(), sizeof(RsBatchJob) * jobs.size());
        up(r->job_off, job_off.data(), sizeof(int) * job_off.size());
        up(djobs, index.data(), sizeof(RsIndexJob) * slot);
        JPCG_HIP(hipMemsetAsync(r->exported, 0, sizeof(unsigned) * bits, st));
        JPCG_HIP(hipMemsetAsync(dflag, 0, sizeof(int), st));
        launch_rs_index(st, djobs, slot, m.rowptr, m.col, hcap, r->hcol, r->hcount, r->lidx, r->exported, dflag);
        std::vector<int> hcount(slot);
        int flag = 0;
        JPCG_HIP(hipMemcpyAsync(hcount.data(), r->hcount, sizeof(int) * slot, hipMemcpyDeviceToHost, st));
        JPCG_HIP(hipMemcpyAsync(&flag, dflag, sizeof(int), hipMemcpyDeviceToHost, st));
        JPCG_HIP(hipStreamSynchronize(st));
        (void)hipFree(djobs);
        (void)hipFree(dflag);
        djobs = nullptr;
        dflag = nullptr;
        RsBatchArgs& a = r->args;
        if (!flag) {
            const int halo = *std::max_element(hcount.begin(), hcount.end());
            r->nh = halo <= kBatchHalo * (r->bs - kWave) ? kBatchHalo : kBatchHaloMost;
            r->lds = rs_lds(RS_STANDARD, r->K, r->bs, rows_max, halo, a.common.lds_slots);
        }
        if (flag || r->lds > kRsMaxLds / per_cu) {
            destroy_batch_resident(r);
            return nullptr;
        }
        JPCG_HIP(hipFuncSetAttribute(rs_batch_kernel(r->K, r->bs, r->nh), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)(kRsMaxLds / per_cu)));
        a.sys = r->sys;
        a.jobs = r->jobs;
        a.job_off = r->job_off;
        a.common.rowptr = m.rowptr;
        a.common.lidx = r->lidx;
        a.common.val = m.val;
        a.common.dinv = m.dinv;
        a.common.exported = r->exported;
        a.common.hcol = r->hcol;
        a.common.hcount = r->hcount;
        a.common.hcap = hcap;
        a.common.sums = (char*)r->words;
        a.common.xch = r->words + sw;
        a.common.xch_step = xw;
        a.run.abort = (unsigned*)(a.common.xch + 2 * xw);
        a.gate = a.run.abort + 32;
        a.run.given_up = &r->out[m.nsys].stop;
        a.out = r->out;
        return r;
    } catch (...) {
        if (djobs) (void)hipFree(djobs);
        if (dflag) (void)hipFree(dflag);
        destroy_batch_resident(r);
        if (!out_of_memory()) throw;
        return nullptr;  // the matrices are streamed
    }
}

bool run_batch_resident(cg_batch_resident* r, int device, hipStream_t st, const double* b, double* x, double tol,
                        int maxit, long long limit, const RsOut*& out)
{
    if (!r->retry.now()) return false;
    RsBatchArgs a = r->args;
    a.common.b = b;
    a.common.x = x;
    a.run.tol = tol;
    a.run.drop2 = 0.0;
    a.run.maxit = maxit;
    // A system's first round lasts as long as its workgroups' earlier systems
    // take: as all are on the card (the gate) and these end by themselves, in
    // maxit iterations or by a wait of their own that runs out, its limit is
    // above what all systems' iterations can take (100 us each; 6 measured).  The
    // gate waits only as long as a launch does.
    a.run.limit = limit;
    a.gate_limit = limit / 160;
    if (test_hooks().wait_limit >= 0) a.run.limit = test_hooks().wait_limit;
    const long long iterations = maxit > 0 ? (long long)maxit * r->nsys : r->rows;
    a.run.limit_first = a.run.limit + iterations * (limit / 80000);
    std::lock_guard<std::mutex> lock(resident_mutex(device));
    for (int s = 0; s < r->nsys; ++s) r->out[s].stop = RS_ABORTED;
    *a.run.given_up = 0;
    launch_rs_clear(st, r->words, r->nwords, nullptr, nullptr, 0);
    void* args[] = {&a};
    JPCG_HIP(hipLaunchKernel(rs_batch_kernel(r->K, r->bs, r->nh), dim3(r->grid), dim3(r->bs), args, r->lds, st));
    JPCG_HIP(hipStreamSynchronize(st));
    if (test_hooks().given_up) *a.run.given_up = 1;
    out = r->out;
    bool ok = *a.run.given_up == 0;
    for (int s = 0; s < r->nsys; ++s) ok = ok && out[s].stop != RS_ABORTED;
    r->retry.done(ok);
    return ok;
}

}  // namespace jpcg
