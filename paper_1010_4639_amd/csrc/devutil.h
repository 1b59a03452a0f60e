// Device helpers shared by the kernel files: XCD-aware workgroup order and
// deterministic (fixed-tree) reductions.
#pragma once

#include <hip/hip_runtime.h>

#include "plan.h"

namespace cgmi {
namespace dev {

constexpr int kWaves = kBlock / 64;
constexpr int kXcds = 8; // MI355X: workgroups are dealt round-robin to 8 XCDs, each with its own L2

// Workgroup id -> logical chunk, so that each XCD works on one contiguous
// range of chunks (neighbouring rows share x and y lines in that XCD's L2).
__device__ __forceinline__ int xcd_remap(int bid, int nblk)
{
    const int per = nblk / kXcds, rem = nblk % kXcds;
    const int x = bid % kXcds, i = bid / kXcds;
    return x * per + min(x, rem) + i;
}

// x[c] for c >= 0, else 0.  FP32 x: the load is unguarded (index clamped to
// 0; x holds at least one element) and the value selected, since a guarded
// load takes its conversion to FP64 into the branch and waits there,
// serialising the gathers of a round.  FP64 x: a guarded load (nothing to
// convert; the unguarded form costs address registers and occupancy).
template <class PT>
__device__ __forceinline__ PT gather0(const PT *__restrict__ x, int c)
{
    if constexpr (sizeof(PT) == 4) {
        const PT v = x[c < 0 ? 0 : c];
        return c >= 0 ? v : PT(0);
    } else {
        return c >= 0 ? x[c] : PT(0);
    }
}

// Store of a value that a later kernel reads: through the XCD's L2 to memory
// at once (an agent-scope store), so the lines are clean when the kernel ends
// and its write-back has nothing left to do, and the writes of a streaming
// kernel leave in step with its reads.  160^3 CSR iteration, all vector
// stores: 175.0 -> 171.8 us (product 126.4 -> 124.3); 61x59x57: 14.5 -> 14.1.
template <class T>
__device__ __forceinline__ void store_through(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// v of the lane `R` places further round its row of 16 lanes (a vector
// register move, where a shuffle goes through the LDS unit).
template <int R>
__device__ __forceinline__ double row_rotate(double v)
{
    const int64_t b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x120 + R, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x120 + R, 0xf, 0xf, true);
    return __longlong_as_double((int64_t)hi << 32 | (uint32_t)lo);
}

// v + its partner's v across the halves of the wavefront (H = 32) or of each
// half (H = 16): the swap of the odd halves of one copy with the even ones of
// another leaves both addends in every lane.
template <int H>
__device__ __forceinline__ double half_sum(double v)
{
    const int64_t b = __double_as_longlong(v);
    unsigned l0, l1, h0, h1;
    if constexpr (H == 32) {
        const auto l = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
        l0 = l[0], l1 = l[1], h0 = h[0], h1 = h[1];
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
        l0 = l[0], l1 = l[1], h0 = h[0], h1 = h[1];
    }
    return __longlong_as_double((int64_t)((uint64_t)h0 << 32 | l0)) +
           __longlong_as_double((int64_t)((uint64_t)h1 << 32 | l1));
}

// Butterfly sum over groups of W lanes: every lane of the group holds the same
// bits.  A whole wavefront (all lanes active) adds partners 32, 16, 8, ... 1
// lanes apart without the LDS unit: after the steps before it, the value 8, 4,
// 2 or 1 lanes round a row of 16 is the partner's.  (By shuffles every
// reduction of an iteration waited for six round trips to the LDS unit:
// iteration of 205 143 rows 14.15 -> 13.4 us, of 100^3 39.2 -> 38.2.)
template <int W>
__device__ __forceinline__ double group_sum(double v)
{
    if constexpr (W == 64) {
        v = half_sum<32>(v);
        v = half_sum<16>(v);
        v += row_rotate<8>(v);
        v += row_rotate<4>(v);
        v += row_rotate<2>(v);
        v += row_rotate<1>(v);
        return v;
    }
#pragma unroll
    for (int o = W / 2; o > 0; o >>= 1)
        v += __shfl_xor(v, o, W);
    return v;
}

// Sum over a workgroup of TB threads (red: TB / 64 entries); every thread
// returns the same bits.  Waves are added in index order, so waves whose
// threads all hold +0.0 leave the bits of the sum over the others unchanged.
template <int TB>
__device__ __forceinline__ double block_sum_n(double v, double *red)
{
    v = group_sum<64>(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = red[0];
#pragma unroll
    for (int w = 1; w < TB / 64; ++w)
        t += red[w];
    return t;
}

// Sum over the workgroup; every thread returns the same bits.
__device__ __forceinline__ double block_sum(double v, double *red)
{
    v = group_sum<64>(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = red[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w)
        t += red[w];
    return t;
}

// Partials (m <= N * kBlock) in two steps, so that their loads can be
// issued before a kernel's own loads and summed while those are in flight:
// partials_load, then partials_sum, which adds them in the order of
// reduce_partials (same bits).
constexpr int kPartPerThread = (kMaxSpmvBlocks + kBlock - 1) / kBlock;
static_assert(kMaxVecBlocks <= kMaxSpmvBlocks, "vector partials fit the same registers");

template <int N>
__device__ __forceinline__ void partials_load(const double *__restrict__ part, int m, double (&pv)[N])
{
    // unguarded loads (index clamped to m - 1, m >= 1) and a select: a
    // guarded load would take the first add of the sum into its branch and
    // wait there before the next load is issued
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int i = threadIdx.x + j * kBlock;
        const double v = part[min(i, m - 1)];
        pv[j] = i < m ? v : 0.0;
    }
}

template <int N>
__device__ __forceinline__ double partials_sum(const double (&pv)[N], int m, double *red)
{
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < N; ++j)
        if ((int)threadIdx.x + j * kBlock < m)
            s += pv[j];
    return block_sum(s, red);
}

// Sum of m per-workgroup partials, identical in every workgroup.
__device__ __forceinline__ double reduce_partials(const double *__restrict__ part, int m, double *red)
{
    double s = 0.0;
    for (int i = threadIdx.x; i < m; i += kBlock)
        s += part[i];
    return block_sum(s, red);
}

} // namespace dev
} // namespace cgmi
