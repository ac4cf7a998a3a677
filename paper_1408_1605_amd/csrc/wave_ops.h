// Wave64 and workgroup primitives (device code).
#pragma once

#include "bfs_internal.h"

namespace bfsmi {

// Number of set bits of mask in lanes below the calling lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Waits until this wave's stores and atomics have reached the L2 (or with
// device scope the other XCDs).  The signal fences, no instructions
// themselves, keep the compiler from moving a store across the wait.
__device__ __forceinline__ void wait_stores()
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T x)
{
    const int lane = __lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const T y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// Inclusive scan of a 32-bit value over the wave by DPP row shifts and
// broadcasts (a few cycles a step, where a shuffle goes through the LDS).
// Every lane of the wave must be active.
__device__ __forceinline__ int32_t wave_inclusive_scan_dpp(int32_t x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return x;
}

// As wg_exclusive_scan below, for 32-bit values, with DPP steps in the wave.
__device__ __forceinline__ uint32_t wg_exclusive_scan_dpp(uint32_t x, uint32_t* total,
                                                          uint32_t* s_wave)
{
    const int lane = __lane_id();
    const int wave = threadIdx.x >> 6;
    const uint32_t incl = (uint32_t)wave_inclusive_scan_dpp((int32_t)x);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kWG / 64; ++w) {
        const uint32_t t = s_wave[w];
        if (w < wave) before += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return before + incl - x;
}

// Exclusive scan over the 256 threads of a workgroup; *total receives the
// sum.  s_wave must hold kWG / 64 elements.  Contains two barriers: every
// thread of the workgroup must call it.
template <typename T>
__device__ __forceinline__ T wg_exclusive_scan(T x, T* total, T* s_wave)
{
    const int lane = __lane_id();
    const int wave = threadIdx.x >> 6;
    const T incl = wave_inclusive_scan(x);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    T before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kWG / 64; ++w) {
        const T t = s_wave[w];
        if (w < wave) before += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return before + incl - x;
}

// The 32 flag bytes (0 or 1) of word w's ids as bits.
__device__ __forceinline__ uint32_t flag_bits(const uint4* found16, int64_t w)
{
    const uint4 x = found16[2 * w], y = found16[2 * w + 1];
    const uint32_t q[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
    uint32_t pf = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t z = q[k];
        pf |= ((z & 1u) | ((z >> 7) & 2u) | ((z >> 14) & 4u) | ((z >> 21) & 8u)) << (4 * k);
    }
    return pf;
}

}  // namespace bfsmi
