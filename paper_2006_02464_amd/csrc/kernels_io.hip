// OUTPUT: results into pinned host memory, and the wait for an EXEC of another stream.
#include "conv_common.h"

namespace cw {

// OUTPUT's copies as one launch: row y of the grid writes the probabilities (0) or the logits (1) into the caller's pinned memory,
// 16 bytes a lane, past the caches.  Bound: the launch (at most 128 KB in the usual batches).  As two copies of the runtime the
// second began 10 to 20 us behind the first; a request alone on the GPU, Inception 127x127 batch 5 189 -> 155..168 us, MobileNet
// batch 16 447 -> 415..428; among others 120.5 -> 115 and 252 -> 254, ResNet-18 64x64 batch 8 127 -> 106.  (INPUT's copy stays with
// the runtime's copy engines: 16 workgroups read pinned memory at the same 57 GB/s, but whatever shares their CUs then waits
// for PCIe in the same load path: MobileNet batch 16 253 -> 347 us.)
__global__ __launch_bounds__(256) void copy_out_kernel(const void *probs, void *host_probs, const void *logits, void *host_logits, unsigned words) {
    constexpr int kSystemScope = 17;   // cache-policy operand: sc0 sc1
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(blockIdx.y ? logits : probs, words * 4u), rd = make_rsrc(blockIdx.y ? host_logits : host_probs, words * 4u);
    const unsigned n = blockIdx.x * 256u + threadIdx.x, step = gridDim.x * 1024u, whole = words & ~3u;
    for (unsigned w = n * 4u; w < whole; w += step)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_amdgcn_raw_buffer_load_b128(rs, w * 4u, 0, 0), rd, w * 4u, 0, kSystemScope);
    if (n < words - whole) __builtin_amdgcn_raw_buffer_store_b32(__builtin_amdgcn_raw_buffer_load_b32(rs, (whole + n) * 4u, 0, 0), rd, (whole + n) * 4u, 0, kSystemScope);
}

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

hipError_t launch_copy_out(void *host_probs, const void *probs, void *host_logits, const void *logits, size_t bytes, hipStream_t s) {
    if (bytes == 0 || bytes % 4 != 0 || bytes >= (1ull << 31) || !host_probs) return hipErrorInvalidValue;
    const size_t wgs = (bytes + 4095) / 4096;
    copy_out_kernel<<<dim3((unsigned)(wgs < 64 ? wgs : 64), host_logits ? 2 : 1), 256, 0, s>>>(probs, host_probs, logits, host_logits, (unsigned)(bytes / 4));
    return hipGetLastError();
}

hipError_t launch_wait_done(const unsigned *done, unsigned seq, unsigned us, hipStream_t s) {
    if (!done || us > 1000000) return hipErrorInvalidValue;
    wait_done_kernel<<<1, 64, 0, s>>>(done, seq, us * 100);
    return hipGetLastError();
}

}  // namespace cw
