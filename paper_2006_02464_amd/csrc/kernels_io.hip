// The wait of OUTPUT and INPUT for an EXEC of another stream.
#include "common.h"

namespace cw {

// A queue of the GPU whose next packet waits for a signal makes every launch of the other queues about 1 us longer; a queue that
// runs a sleeping wave does not.  A stream that is about to wait for an EXEC therefore runs this first: it ends as the EXEC's
// softmax begins, or after `ticks`, and the wait behind it is short.  INPUT, EXEC and OUTPUT on streams of their own, us a request:
// ResNet-18 64x64 batch 1 116 -> 97, ResNet-50 batch 4 336 -> 295 (EXEC alone 272), Inception 127x127 batch 5 125 -> 121, MobileNet
// batch 16 257 -> 253.
__global__ __launch_bounds__(64) void wait_done_kernel(const unsigned *done, unsigned seq, unsigned ticks) {
    const unsigned long long from = __builtin_amdgcn_s_memrealtime();   // 100 MHz
    while ((int)(__hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - seq) < 0 && __builtin_amdgcn_s_memrealtime() - from < ticks)
        __builtin_amdgcn_s_sleep(8);   // 512 clocks
}

hipError_t launch_wait_done(const unsigned *done, unsigned seq, unsigned us, hipStream_t s) {
    if (!done || us > 1000000) return hipErrorInvalidValue;
    wait_done_kernel<<<1, 64, 0, s>>>(done, seq, us * 100);
    return hipGetLastError();
}

}  // namespace cw
