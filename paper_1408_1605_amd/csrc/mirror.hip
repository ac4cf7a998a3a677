// Reading control words back to the host.
//
// A level loop that the host drives reads a few words after every level.  As a
// device-to-host copy and a stream synchronisation that took 20 to 30 us per
// level (a copy kernel, its packet, the runtime's wait), more than most levels
// of a small graph.  Here the device stores the words into pinned host memory
// itself, with a sequence number behind them, and the host polls that number:
// one search of R-MAT 16 236 -> 200 us, R-MAT 22 697 -> 656, the
// 2x4 blocked search of R-MAT 20 1163 -> 1112 (its plan also travels as a kernel
// argument instead of a copy).
#include <hip/hip_runtime.h>

#include <chrono>

#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#include <immintrin.h>
#endif

#include "runtime.h"

namespace bfsmi {

// One wave copies n16 16-byte words to dst (pinned host memory), then stores
// seq behind them.
__global__ __launch_bounds__(64) void k_publish(const int4* __restrict__ src, int32_t n16,
                                                int4* __restrict__ dst, uint64_t* __restrict__ flag,
                                                uint64_t seq)
{
    for (int i = threadIdx.x; i < n16; i += 64) dst[i] = src[i];
    __threadfence_system();
    if (threadIdx.x == 0)
        __hip_atomic_store(flag, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_publish(hipStream_t s, const void* src, size_t bytes, void* dst, uint64_t* flag,
                          uint64_t seq)
{
    if (bytes % 16) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, static_cast<const int4*>(src),
                       (int32_t)(bytes / 16), static_cast<int4*>(dst), flag, seq);
    return hipGetLastError();
}

int wait_published(const uint64_t* flag, uint64_t seq, hipStream_t s)
{
    // polls for as long as a level usually takes, then leaves the wait (and
    // the report of a device error) to the runtime
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t i = 1;; ++i) {
        if (__atomic_load_n(flag, __ATOMIC_ACQUIRE) == seq) return BFS_OK;
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
        _mm_pause();
#endif
        if (i % 256 == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(500)) break;
    }
    BFS_HIP_TRY(hipStreamSynchronize(s));
    if (__atomic_load_n(flag, __ATOMIC_ACQUIRE) != seq)
        return fail(BFS_ERR_HIP, "the device did not publish its control block");
    return BFS_OK;
}

}  // namespace bfsmi
