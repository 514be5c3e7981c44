// Device and host helpers shared by the solver kernels (gfx950, wave64).
//
// Everything reduces in a fixed order: a wave reduces by pairwise exchanges
// (each lane adds its partner's value, and IEEE addition is commutative, so
// both partners, and in the end every lane, hold the same bits), a block adds
// its waves in index order, and a grid reduction adds per-block partials in a
// fixed strided order followed by the same block reduction.
// Repeated runs with the same launch shape are therefore bitwise identical,
// and every block that reduces the same partials obtains the same scalar,
// which keeps the control flow of all blocks in step.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <string>

#include "../../include/jpcg.h"

namespace jpcg {

constexpr int kWave = 64;

// ---------------------------------------------------------------------------
// Reductions
// ---------------------------------------------------------------------------
template <int WIDTH, typename T>
__device__ __forceinline__ T group_sum(T v)
{
    // Butterfly within aligned groups of WIDTH lanes (WIDTH a power of two <= 64).
#pragma unroll
    for (int off = WIDTH / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Sum of a double over the 64 lanes of a fully active wave, the same bits in
// every lane.  Within each row of 16 lanes four DPP exchanges pair lane i with
// i ^ 1, i ^ 2, 7 - i (within 8) and 15 - i: after each, the lanes of the
// pairs merged so far hold one value, so the next exchange adds two equal
// groups.  The four row sums are then read as scalars (lanes 0, 16, 32, 48)
// and added as (r0 + r1) + (r2 + r3).  DPP moves run in the vector ALU, not
// through the LDS crossbar that a lane shuffle takes.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, (unsigned long long)(unsigned)lo | ((unsigned long long)(unsigned)hi << 32));
}

__device__ __forceinline__ double read_lane(double v, int lane)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
}

template <int K>
__device__ __forceinline__ void wave_sum(double (&v)[K])
{
    constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kRowHalfMirror = 0x141, kRowMirror = 0x140;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += dpp_move<kQuadXor1>(v[k]);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += dpp_move<kQuadXor2>(v[k]);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += dpp_move<kRowHalfMirror>(v[k]);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += dpp_move<kRowMirror>(v[k]);
#pragma unroll
    for (int k = 0; k < K; ++k)
        v[k] = (read_lane(v[k], 0) + read_lane(v[k], 16)) + (read_lane(v[k], 32) + read_lane(v[k], 48));
}

// Sum K values over the block; the totals are returned in every thread.
// `lds` must hold (BS / 64) * K doubles.
template <int BS, int K>
__device__ __forceinline__ void block_sum(double (&v)[K], double* lds)
{
    constexpr int NW = BS / kWave;
    const int w = threadIdx.x / kWave, l = threadIdx.x % kWave;
    wave_sum<K>(v);
    __syncthreads();
    if (l == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) lds[w * K + k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < NW; ++j) s += lds[j * K + k];
        v[k] = s;
    }
}

// Write the block's K partial sums to part[slot * K + k] (interleaved, so a
// reader fetches one block's K values with one vector load).
template <int BS, int K>
__device__ __forceinline__ void block_partials(double (&v)[K], double* lds, double* part, int slot)
{
    block_sum<BS, K>(v, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) part[slot * K + k] = v[k];
    }
}

// Every block reduces the G interleaved K-tuples of partials in the same
// order, so every block obtains the same bits.
template <int BS, int K>
__device__ __forceinline__ void grid_sum(const double* part, int G, double (&out)[K], double* lds)
{
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = 0.0;
    for (int j = threadIdx.x; j < G; j += BS) {
#pragma unroll
        for (int k = 0; k < K; ++k) out[k] += part[j * K + k];
    }
    block_sum<BS, K>(out, lds);
}

// Every WAVE reduces the G interleaved K-tuples itself: lane l adds entries
// l, l+64, ... in order, then pairwise lane exchanges give every lane the same
// bits (wave_sum).  No LDS and no workgroup barrier, so the loads can overlap
// other work issued before the first use of the result.
template <int K>
__device__ __forceinline__ void wave_grid_sum(const double* __restrict__ part, int G, double (&out)[K])
{
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = 0.0;
#pragma unroll 4
    for (int j = lane; j < G; j += kWave) {
#pragma unroll
        for (int k = 0; k < K; ++k) out[k] += part[j * K + k];
    }
    wave_sum<K>(out);
}

// ---------------------------------------------------------------------------
// Grid barrier for co-resident (cooperatively launched) grids.
//
// Sense by generation: each arriving block adds one to `count`, which only
// grows during a launch (it is cleared before the launch); the block whose
// arrival completes generation g (count reaching (g + 1) * nblocks) advances
// `gen`, and the others spin on `gen`.  Never resetting `count` matters: a
// reset store and the `gen` store may become visible in either order, and a
// fast block's arrival at the next barrier could then be wiped out.  Thread 0
// of a block fences at agent scope before arriving (publishing the block's
// writes to all XCDs) and after leaving (so later loads observe other blocks'
// writes).  Every wait is bounded by a wall-clock limit: on expiry the block
// raises `abort`, and every waiter that sees `abort` leaves, so all waves
// exit even if a block never arrives.
// ---------------------------------------------------------------------------
struct alignas(256) GridBarrier {
    unsigned count;
    unsigned pad0[63];
    unsigned gen;
    unsigned pad1[63];
    unsigned abort;
    unsigned pad2[63];
};

__device__ __forceinline__ unsigned barrier_gen(GridBarrier* gb)
{
    return __hip_atomic_load(&gb->gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
}

// Returns false if the barrier was abandoned.  `gen` is the block's copy of
// the generation counter; it is advanced on success.  Ordering: a release
// fence before arriving, relaxed atomics and a relaxed spin (an acquiring
// load would invalidate caches on every poll), an acquire-release fence in
// the last arriver before it advances `gen`, and an acquire fence after the
// wait.
__device__ __forceinline__ bool grid_barrier(GridBarrier* gb, unsigned nblocks, unsigned& gen,
                                             long long limit_ticks, int* s_flag)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        int ok = 1;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const unsigned prev = __hip_atomic_fetch_add(&gb->count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == (gen + 1) * nblocks - 1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
            __hip_atomic_store(&gb->gen, gen + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            const long long t0 = wall_clock64();
            while (__hip_atomic_load(&gb->gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gen) {
                __builtin_amdgcn_s_sleep(1);
                if (__hip_atomic_load(&gb->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    ok = 0;
                    break;
                }
                if (wall_clock64() - t0 > limit_ticks) {
                    __hip_atomic_store(&gb->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ok = 0;
                    break;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *s_flag = ok;
    }
    __syncthreads();
    const bool ok = *s_flag != 0;
    gen += 1;
    __syncthreads();  // s_flag may be rewritten by the next barrier
    return ok;
}

// Map the hardware block index to a logical one so that the blocks that land
// on one XCD (dispatched round-robin, block b on XCD b % 8) own a contiguous
// range of rows and share gathered vector entries in that XCD's L2.
__device__ __forceinline__ int xcd_logical_block(int b, int G)
{
    constexpr int kXcd = 8;
    if (G % kXcd != 0) return b;
    return (b % kXcd) * (G / kXcd) + b / kXcd;
}

// ---------------------------------------------------------------------------
// Host helpers
// ---------------------------------------------------------------------------
struct HipError {
    hipError_t code;
    const char* what;
};

#define JPCG_HIP(call)                                             \
    do {                                                           \
        hipError_t e_ = (call);                                    \
        if (e_ != hipSuccess) throw ::jpcg::HipError{e_, #call};   \
    } while (0)

// In a handler: whether the exception is device memory running out (HIP's own
// record of the error is then cleared).
inline bool out_of_memory()
{
    try {
        throw;
    } catch (const HipError& e) {
        if (e.code != hipErrorOutOfMemory) return false;
        (void)hipGetLastError();
        return true;
    } catch (...) {
        return false;
    }
}

}  // namespace jpcg
