// A whole CG solve in one kernel, with the matrix and every vector on chip.
//
// The 256 compute units of the card hold 128 MB of registers; a system whose
// rows fit one row to a thread (up to 1024 rows per workgroup, one workgroup
// per compute unit) is read from memory once per solve: each thread keeps its
// row's values, its row's column slots (indices into the workgroup's LDS
// vector) and its entries of x, r, p, z and the Jacobi diagonal in registers.
// An iteration then moves only what crosses workgroups: the entries of one
// vector that other workgroups' rows refer to (the "halo") and the partial
// sums of the dot products.
//
// Both are exchanged through memory without barriers, fences or atomic read-
// modify-writes: a double travels as two 8-byte words, each carrying 32 bits
// of the value and a 32-bit tag (the round's number).  A reader polls until
// both words carry the round's tag, so every word says by itself whether it is
// the one awaited and no order between different words is relied on.  Two
// buffers by the tag's parity suffice: a workgroup writes round t + 2 only
// after round t + 1 has brought it every workgroup's sums, and those are
// published after round t has been read.  The buffers are cleared by a kernel
// of their own before each solve (tag 0 is never awaited).
//
// Measured between two workgroups, one way: 0.27 us through the L2 of one XCD
// (plain store, sc1 load), 0.55-0.67 us between XCDs (sc1 store and load).
// 256 workgroups polling each other's 256 sums take several times that, so
// sums go in two stages: the workgroups of a group (the blocks that land on
// one XCD, at most 32) read each other's through their L2, and one of each
// group publishes the group's sum for all.  A system that fits one XCD's
// compute units uses one group and never leaves its L2.  Halo entries that
// only the own group reads stay in its L2 too.  Whether a group's workgroups
// do sit on one XCD is asked of the hardware at the start of each solve; if
// not, the group's stores are written through like the others.  Groups own
// whole 128-byte lines of the exchanged vector, so no line is written through
// two L2s.
//
// Every workgroup adds the same sums in the same order, so all of them reach
// the same bits and take the same branches.  Every wait is bounded: a
// workgroup that waits too long raises an abort word and leaves, and so do all
// that wait in vain for it.  Others may have seen what it did not and finish
// the solve, so the host takes no result of a launch in which any workgroup
// gave up: x is put back and the kernels of std_kernels.hpp, sr_kernels.hpp or
// ell_kernels.hpp solve the system.
//
// What bounds it: the latency of the rounds, two an iteration in the standard
// form and one in the single-reduction form, each a chain of LDS, cross-lane
// and exchange latencies; the product itself is 27 LDS reads a row.  Time per
// iteration against the graph-chunked kernels', N rows of 27 nonzeros:
//   N = 4096 (one group)      2.9 us against 13.0 (single-reduction 2.8)
//   N = 132651 (eight groups) 5.2 us against 18.5 (single-reduction 5.2)
// of which the two rounds' sums take 1.2 us within one XCD and 3.4 us across
// eight.  With all 256 workgroups polling each other's sums directly the
// iteration took 10.4 us (8.8 with pauses between the polls).
#pragma once

#include <type_traits>

#include "phases.hpp"

namespace jpcg {

using u64 = unsigned long long;

// The most sums exchanged in a round, workgroups of a group, XCDs, and groups
// of a team (two on an XCD where workgroups run two to a compute unit).
constexpr int kRsSums = 5;
constexpr int kRsGroup = 32;
constexpr int kRsXcds = 8;
constexpr int kRsGroups = 16;
// Bytes of a team's sums for one parity: [group][sum][member] of 16 bytes, and
// a line of 128 bytes per group with its sums.
constexpr unsigned kRsSumBytes = kRsGroups * (16u * kRsSums * kRsGroup + 128u);
__device__ __forceinline__ unsigned rs_member_sum(int group, int sum, int member)
{
    return 16u * (unsigned)((group * kRsSums + sum) * kRsGroup + member);
}
__device__ __forceinline__ unsigned rs_group_sum(int sum, int group)
{
    return 16u * (unsigned)(kRsGroups * kRsSums * kRsGroup) + 128u * (unsigned)group + 16u * (unsigned)sum;
}
// Vectors kept for the halo columns: p, or d, r and s (single-reduction form).
constexpr int kRsHaloState = 3;
constexpr int kRsMaxSlot = 0x7fffffff;
// Blocks whose threads have 128 registers: 1024 threads, or 512 two to a
// compute unit.
constexpr bool rs_tight(int bs) { return bs == 1024 || bs == 512; }

struct RsOut {
    int stop, iters, replacements, pad;
    double nb, rr, rr_true;
};
constexpr int RS_ABORTED = -1;

// One system as a team of workgroups sees it.  Rows and columns are global
// (a batch is one block-diagonal matrix); the system's rows start at row0.
struct RsSys {
    int row0, n;
    int groups, members;  // of the team; workgroups = groups * members
    int rpw;              // rows per workgroup, a multiple of 8
    const int* rowptr;
    const unsigned short* lidx;  // per nonzero: slot of its column in the workgroup's LDS vector
    const double* val;
    const float* val32;     // FP32-matrix form
    const double* rowsum;   // FP32-matrix form
    const double* dinv;
    const unsigned* exported;  // bit per row of the system: read outside its group
    const int* hcol;        // [G][hcap]: columns of each workgroup's halo, from row0
    const int* hcount;      // [G]
    int hcap;
    int lds_slots;          // where the columns' offsets start in LDS, in doubles
    const double* b;
    double* x;
    u64* xch;               // two words per row of the system; odd rounds' xch_step words on
    size_t xch_step;
    char* sums;             // kRsSumBytes; odd rounds' as many bytes on
    RsOut* out;
    double* hist;
};

struct RsRun {
    double tol, drop2;  // drop2 > 0: the FP32-matrix form's reliable updates (see CgArgsT)
    int maxit;
    unsigned* abort;    // raised for the other workgroups
    int* given_up;      // and for the host (pinned)
    // Bounds of a wait, device wall clock ticks: until a solve's first round has
    // brought every workgroup's sums, and from then on.
    long long limit_first, limit;
};

// A double in flight: two 8-byte words, each with its tag, loaded and stored
// with one 16-byte access at agent scope (sc1: past the caches that other
// XCDs' stores do not reach).  Each word is validated by its own tag.
typedef unsigned rs_words __attribute__((ext_vector_type(4)));  // {low, tag, high, tag}
constexpr int kRsAgent = 16;  // sc1

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rs_buffer(const void* base)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0xffffffffu, 0x00020000);
}

__device__ __forceinline__ rs_words rs_load(__amdgpu_buffer_rsrc_t buf, unsigned byte)
{
    return __builtin_amdgcn_raw_buffer_load_b128(buf, byte, 0, kRsAgent);
}

// `near`: for readers on the same XCD only, whose loads find it in their L2.
__device__ __forceinline__ void rs_publish(__amdgpu_buffer_rsrc_t buf, unsigned byte, double v, unsigned tag, bool near)
{
    const u64 b = __builtin_bit_cast(u64, v);
    const rs_words w{(unsigned)b, tag, (unsigned)(b >> 32), tag};
    if (near) __builtin_amdgcn_raw_buffer_store_b128(w, buf, byte, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b128(w, buf, byte, 0, kRsAgent);
}

// A value that is the same in every lane, kept in scalar registers.
__device__ __forceinline__ double rs_uniform(double v) { return read_lane(v, 0); }

__device__ __forceinline__ double rs_value(rs_words w)
{
    return __builtin_bit_cast(double, (u64)w.x | ((u64)w.z << 32));
}
__device__ __forceinline__ bool rs_tagged(rs_words w, unsigned tag) { return w.y == tag && w.w == tag; }

// The calling workgroup leaves before the end: the others and the host are told.
__device__ __forceinline__ void rs_give_up(const RsRun& run)
{
    __hip_atomic_store(run.abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(run.given_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A bounded wait: true while it may go on.  Past its limit it allows one more
// look.  What is missing in that look may come right after it and be seen by
// the other workgroups, so whether one gave up says nothing about the others:
// only the host decides, by given_up.
struct RsWait {
    const RsRun& run;
    long long limit, t0;
    int spins;
    bool last;
    __device__ __forceinline__ RsWait(const RsRun& r, long long l) : run(r), limit(l), t0(0), spins(0), last(false) {}
    __device__ __forceinline__ bool more()
    {
        if (last) {
            rs_give_up(run);
            return false;
        }
        if ((++spins & 31) != 0) return true;
        const long long now = wall_clock64();
        if (spins == 32) t0 = now;
        last = now - t0 > limit || __hip_atomic_load(run.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
        return true;
    }
};

// Sums over each half of a wave (32 lanes): complete in lanes 16-31 and 48-63.
// `row` alone leaves each lane the sum of its 16 lanes.
__device__ __forceinline__ double rs_row_sum(double v)
{
    v += dpp_move<0xB1>(v);   // lane ^ 1
    v += dpp_move<0x4E>(v);   // lane ^ 2
    v += dpp_move<0x141>(v);  // mirrored in 8
    v += dpp_move<0x140>(v);  // mirrored in 16
    return v;
}
__device__ __forceinline__ double rs_half_sum(double v)
{
    v = rs_row_sum(v);
    // Lane 15 of rows 0 and 2 into rows 1 and 3 (rows 0 and 2 add zero).
    const u64 b = __builtin_bit_cast(u64, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x142, 0xA, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x142, 0xA, 0xF, false);
    return v + __builtin_bit_cast(double, (u64)(unsigned)lo | ((u64)(unsigned)hi << 32));
}

// The solve of one system by one workgroup of its team.  K: slots of a row
// (its longest row, rounded up); NH: halo entries per thread at most.
template <int K, int BS, int NH, bool M32>
struct RsTeam {
    static constexpr bool kTight = rs_tight(BS);
    static constexpr int kSlotWords = kTight ? 2 : K / 2;
    // With 128 registers a thread the columns' offsets and the halo's p stay in
    // LDS, and a product reads fewer entries ahead.  Held in registers they
    // spilled (90 of them): 8.6 us per iteration at 60^3 against 6.2, 6.8
    // against 5.7 in the single-reduction form.
    using VT = std::conditional_t<M32, float, double>;

    const RsSys& s;
    const RsRun& run;
    const int L;
    double* pl;    // LDS: [rows of the workgroup][halo][zero]
    double* hs;    // LDS: [halo] times kRsHaloState, what an iteration keeps of the halo
    double* red;   // LDS: [kRsSums][BS / 4]
    double* tot;   // LDS: [kRsSums]
    int* fail;     // LDS
    unsigned tag = 0;
    long long limit;

    int group, member, tid, ra, nown, H, nh, row;
    bool local;   // the group's workgroups share an L2
    bool near;    // and only they read this thread's row
    int k0, len;
    VT v[K];
    unsigned c[kSlotWords];  // byte offsets of the columns' LDS slots, two to a word
    unsigned* lc;  // the same in LDS: [K / 4][BS] pairs of words
    unsigned hc[NH];  // halo columns, from row0
    double d, xo;

    __device__ __forceinline__ RsTeam(const RsSys& sys, const RsRun& r, int index, double* lds, double* rd, double* t,
                                      int* f)
        : s(sys), run(r), L(index), pl(lds), red(rd), tot(t), fail(f), limit(r.limit_first)
    {
        tid = threadIdx.x;
        group = L / s.members;
        member = L - group * s.members;
        const int first = min(L * s.rpw, s.n);
        nown = min(s.rpw, s.n - first);
        ra = s.row0 + first;
        H = s.hcount[L];
        nh = (H + kHaloThreads - 1) / kHaloThreads;
        row = has() ? ra + tid : s.row0;
        k0 = s.rowptr[row];
        len = has() ? s.rowptr[row + 1] - k0 : 0;
        const unsigned zero = 8u * (unsigned)(nown + H);
        hs = pl + nown + H + 1;
        lc = (unsigned*)(lds + s.lds_slots);
#pragma unroll
        for (int j = 0; j < K; j += 2) {
            const int ka = j < len ? k0 + j : 0, kb = j + 1 < len ? k0 + j + 1 : 0;
            VT va, vb;
            if constexpr (M32) {
                va = s.val32[ka];
                vb = s.val32[kb];
            } else {
                va = s.val[ka];
                vb = s.val[kb];
            }
            const unsigned ca = 8u * s.lidx[ka], cb = 8u * s.lidx[kb];
            v[j] = j < len ? va : VT(0);
            v[j + 1] = j + 1 < len ? vb : VT(0);
            c[j / 2 % kSlotWords] = (j < len ? ca : zero) | ((j + 1 < len ? cb : zero) << 16);
            if (kTight && j % 4 == 2) *(uint2*)(lc + 2 * (j / 4 * BS + tid)) = make_uint2(c[0], c[1]);
            if (j % 4 == 2) __builtin_amdgcn_sched_barrier(0);  // few addresses in registers at a time
        }
#pragma unroll
        for (int j = 0; j < NH; ++j) {
            const int h = halo_slot(j);
            hc[j] = h < H ? (unsigned)s.hcol[(size_t)L * s.hcap + h] : 0u;
        }
        d = s.dinv[row];
        xo = s.x[row];
        local = false;
        near = !(s.exported[(row - s.row0) >> 5] >> ((row - s.row0) & 31) & 1u);
        if (tid == 0) {
            pl[nown + H] = 0.0;
            *fail = 0;
        }
    }

    __device__ __forceinline__ bool has() const { return tid < nown; }

    // The halo entries of a thread.  Wave 0, which adds the sums, has none; the
    // highest waves, which have no rows where the workgroup is not full, take
    // the first.
    static constexpr int kHaloThreads = BS - kWave;
    __device__ __forceinline__ int halo_slot(int j) const
    {
        return tid < kWave ? kRsMaxSlot : (BS - 1 - tid) + kHaloThreads * j;
    }

    __device__ __forceinline__ void publish(double value)
    {
        if (has()) rs_publish(rs_buffer(s.xch + (tag & 1u) * s.xch_step), 16u * (unsigned)(row - s.row0), value, tag,
                              local && near);
    }

    // Halo entries of the vector published in this round.
    __device__ __forceinline__ bool gather(double (&hv)[NH])
    {
        if (nh == 0) return true;
        const auto buf = rs_buffer(s.xch + (tag & 1u) * s.xch_step);
        unsigned need = 0;
#pragma unroll
        for (int j = 0; j < NH; ++j) need |= halo_slot(j) < H ? 1u << j : 0u;
        RsWait wait(run, limit);
        while (need) {
            rs_words got[NH];
            asm volatile("" ::: "memory");  // load again
#pragma unroll
            for (int j = 0; j < NH; ++j)
                if (j < nh) got[j] = rs_load(buf, 16u * hc[j]);
#pragma unroll
            for (int j = 0; j < NH; ++j)
                if (j < nh && (need >> j & 1u) && rs_tagged(got[j], tag)) {
                    hv[j] = rs_value(got[j]);
                    need &= ~(1u << j);
                }
            if (need && !wait.more()) return false;
        }
        return true;
    }

    // Polls one tagged value a lane (lanes with `use`; the others get 0) until
    // every lane has its own.
    __device__ __forceinline__ bool await(const char* base, unsigned byte, bool use, double& v)
    {
        const auto buf = rs_buffer(base);
        RsWait wait(run, limit);
        while (true) {
            asm volatile("" ::: "memory");  // load again
            const rs_words got = rs_load(buf, byte);
            v = use ? rs_value(got) : 0.0;
            if (__ballot(use && !rs_tagged(got, tag)) == 0ull) return true;
            if (!wait.more()) return false;
        }
    }

    // First round: do the group's workgroups sit on one XCD?
    __device__ __forceinline__ bool start()
    {
        if (s.groups * s.members == 1) return true;
        unsigned xcc;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
        ++tag;
        const int lane = tid & (kWave - 1);
        if (tid < kWave) {
            char* const base = s.sums + (tag & 1u) * kRsSumBytes;
            if (lane == 0) rs_publish(rs_buffer(base), rs_member_sum(group, 0, member), (double)xcc, tag, false);
            double id;
            const bool use = lane < s.members;
            const bool ok = await(base, rs_member_sum(group, 0, use ? lane : 0), use, id);
            const bool one = __ballot(use && id != (double)xcc) == 0ull;
            if (lane == 0) {
                tot[0] = one ? 1.0 : 0.0;
                if (!ok) *fail = 1;
            }
        }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(*fail)) return false;
        local = rs_uniform(tot[0]) != 0.0;
        return true;
    }

    // q becomes the team's sums of Q quantities, the same bits in every thread
    // of every workgroup, together with the halo of the vector published in this round
    // (HALO).  False: the wait was given up.
    template <bool HALO, int Q>
    __device__ __forceinline__ bool round(double (&q)[Q], double (&hv)[NH])
    {
        forget();
        const int lane = tid & (kWave - 1), w = __builtin_amdgcn_readfirstlane(tid / kWave);
#pragma unroll
        for (int k = 0; k < Q; ++k) q[k] += dpp_move<0xB1>(q[k]);
#pragma unroll
        for (int k = 0; k < Q; ++k) q[k] += dpp_move<0x4E>(q[k]);
        if ((tid & 3) == 0) {
#pragma unroll
            for (int k = 0; k < Q; ++k) red[k * (BS / 4) + tid / 4] = q[k];
        }
        __syncthreads();
        // Half a wave per quantity: the workgroup's sum, the group's, the team's.
        bool ok = true;
        if (w < (Q + 1) / 2) {
            const int k = min(2 * w + (lane >> 5), Q - 1), l = lane & 31;
            double v = 0.0;
#pragma unroll
            for (int j = 0; j < BS / 4; j += 32) v += red[k * (BS / 4) + j + l];
            v = rs_half_sum(v);
            if (s.groups * s.members > 1) {
                char* const base = s.sums + (tag & 1u) * kRsSumBytes;
                if (l == 31) rs_publish(rs_buffer(base), rs_member_sum(group, k, member), v, tag, local);
                const bool use = l < s.members;
                ok = await(base, rs_member_sum(group, k, use ? l : 0), use, v);
                v = rs_half_sum(v);
                if (s.groups > 1) {
                    if (l == 31 && member == 0) rs_publish(rs_buffer(base), rs_group_sum(k, group), v, tag, false);
                    const bool every = l >= 16 && l - 16 < s.groups;
                    ok = ok && await(base, rs_group_sum(k, every ? l - 16 : 0), every, v);
                    v = rs_row_sum(v);
                }
            }
            if (l == 31) tot[k] = v;
        }
        if (HALO) ok = gather(hv) && ok;
        if (!ok) *fail = 1;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(*fail)) return false;
#pragma unroll
        for (int k = 0; k < Q; ++k) q[k] = tot[k];
        return true;
    }

    // The thread's row of A times the LDS vector: products rounded on their
    // own and added in stored order, as a sequential CSR row sum.
    __device__ __forceinline__ double product()
    {
#pragma clang fp contract(off)
        repack();
        double t = 0.0;
#pragma unroll
        for (int g = 0; g < K; g += kGroup) {
            double e[kGroup];
            entries(g, e);
            __builtin_amdgcn_sched_barrier(0);  // a group's reads in flight together, and no more registers than that
#pragma unroll
            for (int j = 0; j < kGroup; ++j)
                if (g + j < K) {
                    const double a = (double)v[g + j] * e[j];
                    t = t + a;
                }
            asm volatile("" : "+v"(t));  // the group is added here, not below a later branch
        }
        return t;
    }
    // Entries of the LDS vector read ahead of their use.
    static constexpr int kGroup = kTight ? 4 : 14;
    // The LDS vector's entries for the columns g .. g + kGroup of the row.
    __device__ __forceinline__ void entries(int g, double (&e)[kGroup])
    {
        unsigned o[kGroup / 2];
        if constexpr (kTight) {
            const uint2 two = *(const uint2*)(lc + 2 * (g / 4 * BS + tid));
            o[0] = two.x;
            o[1] = two.y;
        } else {
#pragma unroll
            for (int j = 0; j < kGroup / 2; ++j) o[j] = g / 2 + j < K / 2 ? c[(g / 2 + j) % kSlotWords] : 0u;
        }
#pragma unroll
        for (int j = 0; j < kGroup; ++j)
            if (g + j < K)
                e[j] = *(const double*)((const char*)pl + ((j & 1) ? o[j / 2] >> 16 : o[j / 2] & 0xffffu));
    }
    // Keeps what is cheaply formed from these (unpacked offsets, addresses)
    // from being held in registers across iterations.
    __device__ __forceinline__ void repack()
    {
#pragma unroll
        for (int j = 0; j < kSlotWords; ++j) asm volatile("" : "+v"(c[j]));
        if constexpr (M32) {
#pragma unroll
            for (int j = 0; j < K; ++j) asm volatile("" : "+v"(v[j]));  // their conversions to double
        }
    }
    __device__ __forceinline__ void forget()
    {
#pragma unroll
        for (int j = 0; j < NH; ++j) asm volatile("" : "+v"(hc[j]));
        asm volatile("" : "+v"(tid));
        asm volatile("" : "+v"(row));
    }
    // The same from the FP64 values in memory (the FP32-matrix form's true residual).
    __device__ __forceinline__ double product_fp64()
    {
#pragma clang fp contract(off)
        repack();
        double t = 0.0;
#pragma unroll
        for (int g = 0; g < K; g += kGroup) {
            double e[kGroup];
            entries(g, e);
#pragma unroll
            for (int j = 0; j < kGroup; ++j)
                if (g + j < K) {
                    const double a = (g + j < len ? s.val[k0 + g + j] : 0.0) * e[j];
                    t = t + a;
                }
            asm volatile("" : "+v"(t));
        }
        return t;
    }
    // Row-sum-preserving product of the FP32 values (see tiles.hpp).
    __device__ __forceinline__ double product_diff(double xi)
    {
        repack();
        double t = 0.0;
#pragma unroll
        for (int g = 0; g < K; g += kGroup) {
            double e[kGroup];
            entries(g, e);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < kGroup; ++j)
                if (g + j < K) t = __builtin_fma((double)v[g + j], e[j] - xi, t);
            asm volatile("" : "+v"(t));
        }
        return __builtin_fma(has() ? s.rowsum[row] : 0.0, xi, t);
    }
    // f(j, h) for the thread's halo entries h (its j-th).
    template <typename F>
    __device__ __forceinline__ void each_halo(F f) const
    {
#pragma unroll
        for (int j = 0; j < NH; ++j) {
            const int h = halo_slot(j);
            if (j < nh && h < H) f(j, h);
        }
    }

    // The LDS vector from the thread's own entry and halo entries.
    __device__ __forceinline__ void place(double own, const double (&hv)[NH])
    {
        if (has()) pl[tid] = own;
        each_halo([&](int j, int h) { pl[nown + h] = hv[j]; });
        __syncthreads();
    }

    __device__ __forceinline__ void finish(int stop, int iters, int repl, double nb, double rr, double rrt)
    {
        if (has() && stop != STOP_CONV0) s.x[row] = stop == STOP_ZERO_RHS ? 0.0 : xo;
        if (tid == 0 && L == 0) *s.out = RsOut{stop, iters, repl, 0, nb, rr, rrt};
    }

    // sqrt(rr) <= thr, the root taken only near the threshold.
    __device__ __forceinline__ bool passes(double rr, double thr) const
    {
        return rr <= threshold(thr) && sqrt(rr) <= thr;
    }

    __device__ __forceinline__ void record(int k, double rr, double nb)
    {
        if (s.hist && tid == 0 && L == 0) s.hist[k] = nb > 0.0 ? sqrt(rr) / nb : 0.0;
    }

    // x's halo as the caller passed it, from memory: only before the first
    // round, while x still holds that.
    __device__ __forceinline__ void caller_halo(double (&hv)[NH])
    {
#pragma unroll
        for (int j = 0; j < NH; ++j) hv[j] = s.x[(unsigned)s.row0 + hc[j]];
    }

    // A value that is the same in every lane, in scalar registers where vector
    // registers are short.
    static __device__ __forceinline__ double keep(double v)
    {
        if constexpr (kTight) return rs_uniform(v);
        else return v;
    }

    // Branches on values that are the same in every lane are taken on a ballot:
    // one scalar branch, no masked execution of both sides.
    static __device__ __forceinline__ bool any(bool c) { return __ballot(c) != 0ull; }
    static __device__ __forceinline__ bool positive(double v) { return v > 0.0 && v <= 0x1.fffffffffffffp1023; }

    // Standard form; the order of tests is that of std_kernels.hpp.  The outer
    // loop forms the true residual -- at the start, when the recurrence passes
    // a test, and for the report of a solve that ends without convergence --
    // the inner one iterates.
    __device__ __forceinline__ bool solve_standard()
    {
        double hv[NH] = {};
        double ph[kTight ? 1 : NH] = {};  // the halo's p
        double r, z, p = 0.0, rho = 0.0, beta = 0.0, nb = 0.0, thr = 0.0, rec = 0.0, drop = 0.0, bound = 0.0;
        int k = 0, repl = 0, stop = RUNNING;
        bool begin = true;
        if (!start()) return false;
        caller_halo(hv);
        if constexpr (kTight) each_halo([&](int, int h) { hs[h] = 0.0; });
        while (true) {
            if (!begin) {
                double none[1] = {0.0};
                ++tag;
                publish(xo);
                if (!round<true>(none, hv)) return false;
            }
            place(xo, hv);
            double rr;
            {
                const double bi = has() ? s.b[row] : 0.0;
                double y;
                if constexpr (M32) y = product_fp64();
                else y = product();
                r = has() ? bi - y : 0.0;
                z = d * r;
                double q[3] = {r * z, r * r, bi * bi};
                ++tag;
                publish(z);
                if (!round<true>(q, hv)) return false;
                limit = run.limit;
                rr = q[1];
                if (begin) {
                    nb = rs_uniform(sqrt(q[2]));
                    thr = rs_uniform(run.tol * nb);
                    record(0, rr, nb);
                    if (any(nb == 0.0)) {
                        finish(STOP_ZERO_RHS, 0, 0, nb, rr, 0.0);
                        return true;
                    }
                    if (any(passes(rr, thr))) {
                        finish(STOP_CONV0, 0, 0, nb, rr, rr);
                        return true;
                    }
                    rec = keep(rr);
                    rho = keep(q[0]);
                } else {
                    if (stop != RUNNING) {
                        finish(stop, k, repl, nb, rec, rr);
                        return true;
                    }
                    if (any(passes(rr, thr))) {
                        finish(STOP_CONVERGED, k, repl, nb, rec, rr);
                        return true;
                    }
                    ++repl;
                    record(k, rr, nb);
                    rec = keep(rr);
                    stop = any(!positive(q[0])) ? STOP_BREAKDOWN : k >= run.maxit ? STOP_MAXIT : RUNNING;
                    if (stop != RUNNING) continue;
                    beta = keep(q[0] / rho);
                    rho = keep(q[0]);
                }
                // At or below this ||r||^2 the iteration is left for a test.
                drop = rs_uniform(run.drop2 * rr);
                bound = rs_uniform(fmax(threshold(thr), drop));
            }
            begin = false;
            while (true) {
                // p = z + beta p for the row and, by the same operation as in
                // its owner, for the halo.
                p = __builtin_fma(beta, p, z);
                if constexpr (kTight) {
                    each_halo([&](int j, int h) { hs[h] = hv[j] = __builtin_fma(beta, hs[h], hv[j]); });
                } else {
#pragma unroll
                    for (int j = 0; j < NH; ++j) hv[j] = ph[j] = __builtin_fma(beta, ph[j], hv[j]);
                }
                place(p, hv);
                double ap;
                if constexpr (M32) ap = product_diff(p);
                else ap = product();
                ap = has() ? ap : 0.0;
                double sg[1] = {p * ap};
                ++tag;
                if (!round<false>(sg, hv)) return false;
                if (any(!positive(sg[0]))) {
                    stop = STOP_BREAKDOWN;
                    break;
                }
                const double alpha = rho / sg[0];
                r = __builtin_fma(-alpha, ap, r);
                z = d * r;
                ++tag;
                publish(z);
                xo = __builtin_fma(alpha, p, xo);
                ++k;
                double q[2] = {r * z, r * r};
                if (!round<true>(q, hv)) return false;
                rec = keep(q[1]);
                if (s.hist) record(k, q[1], nb);
                const bool go = q[1] > bound && positive(q[0]);
                if (any(!go) || k >= run.maxit) {
                    // In the order of the tests: residual, r'z, limit.
                    if (any(passes(q[1], thr) || q[1] <= drop)) break;
                    stop = any(!positive(q[0])) ? STOP_BREAKDOWN : k >= run.maxit ? STOP_MAXIT : RUNNING;
                    if (stop != RUNNING) break;
                }
                beta = keep(q[0] / rho);
                rho = keep(q[0]);
            }
        }
    }
    // At or below this ||r||^2, passes() looks closer.
    __device__ __forceinline__ double threshold(double thr) const
    {
        return thr * thr * (1.0 + 0x1p-40) + 0x1p-1060;
    }

    // Single-reduction form (symbols of sr_kernels.hpp): w's halo travels with
    // the sums, and r, s and u of the halo columns are carried here by the
    // operations of their owners.
    __device__ __forceinline__ bool solve_single()
    {
        double hv[NH] = {};
        double r = 0.0, w = 0.0, p = 0.0, sv = 0.0, u = 0.0;
        double nb = 0.0, thr = 0.0, rec = 0.0, gam_old = 0.0, bound = 0.0;
        int k = 0, repl = 0, stop = RUNNING;
        bool begin = true;
        double* const dh = hs;
        double* const rh = hs + H;
        double* const sh = hs + 2 * H;
        if (!start()) return false;
        caller_halo(hv);
        each_halo([&](int j, int h) {
            dh[h] = s.dinv[(unsigned)s.row0 + hc[j]];
            sh[h] = 0.0;
        });
        while (true) {
            // r = b - A x, its test, w = A M^-1 r, and after a replacement
            // s = A p (see k_sr_restart): a product per pass.
            double bi = 0.0;
            for (int pass = 0; pass < 4; ++pass) {
                if (begin && pass == 2) break;  // p = s = 0
                double own = pass == 0 ? xo : pass == 1 ? r : pass == 2 ? p : sv;
                if (!begin || pass > 0) {
                    double q[2] = {r * r, bi * bi};
                    ++tag;
                    publish(own);
                    if (!round<true>(q, hv)) return false;
                    limit = run.limit;
                    if (pass == 1) {
                        if (begin) {
                            rec = keep(q[0]);
                            nb = rs_uniform(sqrt(q[1]));
                            thr = rs_uniform(run.tol * nb);
                            bound = rs_uniform(threshold(thr));
                            record(0, rec, nb);
                            if (any(nb == 0.0)) {
                                finish(STOP_ZERO_RHS, 0, 0, nb, rec, 0.0);
                                return true;
                            }
                            if (any(passes(rec, thr))) {
                                finish(STOP_CONV0, 0, 0, nb, rec, rec);
                                return true;
                            }
                        } else if (stop != RUNNING) {
                            finish(stop, k, repl, nb, rec, q[0]);
                            return true;
                        } else if (any(passes(q[0], thr))) {
                            finish(STOP_CONVERGED, k, repl, nb, rec, q[0]);
                            return true;
                        } else {
                            ++repl;
                        }
                        own = u = d * r;
                        each_halo([&](int j, int h) {
                            rh[h] = hv[j];
                            hv[j] = dh[h] * hv[j];
                        });
                    } else if (pass == 3) {
                        each_halo([&](int j, int h) { sh[h] = hv[j]; });
                        break;
                    }
                }
                place(own, hv);
                double y = product();
                y = has() ? y : 0.0;
                if (pass == 0) {
                    bi = has() ? s.b[row] : 0.0;
                    r = has() ? bi - y : 0.0;
                } else if (pass == 1) {
                    w = y;
                } else {
                    sv = y;
                }
            }
            begin = false;
            while (true) {
                double q[5] = {r * u, w * u, r * r, u * sv + p * w, p * sv};
                ++tag;
                publish(w);
                if (!round<true>(q, hv)) return false;
                const double gam = q[0];
                rec = keep(q[2]);
                if (s.hist) record(k, rec, nb);
                double beta = 0.0, sigma = q[1];
                if (k > 0) {
                    beta = gam / gam_old;
                    sigma = q[1] + beta * q[3] + beta * beta * q[4];
                }
                const bool go = q[2] > bound && positive(gam) && positive(sigma);
                if (any(!go) || k >= run.maxit) {
                    // In the order of the tests: residual, gamma, limit, sigma.
                    if (any(passes(q[2], thr))) break;
                    stop = any(!positive(gam)) ? STOP_BREAKDOWN
                           : k >= run.maxit    ? STOP_MAXIT
                           : any(!positive(sigma)) ? STOP_BREAKDOWN
                                                   : RUNNING;
                    if (stop != RUNNING) break;
                }
                const double alpha = gam / sigma;
                gam_old = keep(gam);
                p = __builtin_fma(beta, p, d * r);
                sv = __builtin_fma(beta, sv, w);
                r = __builtin_fma(-alpha, sv, r);
                u = d * r;
                each_halo([&](int j, int h) {
                    const double s1 = __builtin_fma(beta, sh[h], hv[j]);
                    const double r1 = __builtin_fma(-alpha, s1, rh[h]);
                    sh[h] = s1;
                    rh[h] = r1;
                    hv[j] = dh[h] * r1;
                });
                place(u, hv);
                xo = __builtin_fma(alpha, p, xo);
                w = product();
                w = has() ? w : 0.0;
                ++k;
            }
        }
    }
};

}  // namespace jpcg
